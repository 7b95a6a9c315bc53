// FP6 patch kernel of librmsmp (gfx950): convolutions with filters of several pixels on
// v_mfma_scale_f32_32x32x64_f8f6f4 (fp6_gemm.h has the arithmetic and the operand form of the weights), their input
// widened once and kept in LDS for all taps.
//
// The tile kernel fetches and widens a column for every tap: nine times for a 3x3 layer, and the L1's lookups are what such a layer
// waits for.  Here a work-group stages the input pixels that its output pixels need, one contiguous run of the flattened NHWC
// tensor, as 6-bit operands: 24 bytes per pixel and 32 channels, in two parts, so that a lane's operand of any tap is one 16-byte and one
// 8-byte read at (the lane's pixel + the tap's offset).  Any channel count: a tap's channels are padded to whole blocks of 32
// with zero weights, and what lies there in memory does not matter.  Taps outside the image read a block that holds the zero
// point.
//
// Measured, weights warm, back to back, the kernel that had the layer before / this one: 64 images of a ResNet-18's 3x3 layers, 64 channels of 56 x 56 12.3 / 11.7 us
// (11.3-11.8 / 11.5-11.7 in the benchmark's loop on several cards: no gain), 128 of 28 x 28 12.4 / 10.2, 256 of 14 x 14 11.2 / 10.4 (10.5 / 10.1-10.5), 512 of
// 7 x 7 11.8 / 10.5 (int8, LDS-resident); 144 channels of 16 x 57 x 57 with a bias 18.8 / 13.9 (tile kernel); the heads of 64 and 256 channels with their
// 1x1 layers 12.4 / 12.1 and 12.4 / 8.9.
// What bounds it: a launch is one round of work-groups, each a chain of phases (clock stamps, 128 channels of 28 x 28, 64 x 256 outputs, of
// 18 600 cycles): 500 until the first reads are out, 1 500 more for the weights' first reads, 2 300 until the patch is in LDS, 8 700
// multiplying (5 800 at the matrix cores' rate), 5 400 of vector instructions for the 4-bit codes; and 2 us of launch.  With 32 columns x 2
// a wave the weights' way through the L1 is longer than the products (64 bytes a cycle: 10 700 cycles of 512 channels of 7 x 7, 6 400 without
// these reads): that shape is for grids that fill the chip no other way.
// Waves' code is fetched cold and runs once in front of the K loop, 8 to 10 cycles an instruction, so that part is short: scalar arguments
// in registers, divisions without branches, a column's pixel and taps worked out by one thread for all waves (together 6 700 -> 4 300 cycles).
#pragma once
#include "fp6_gemm.h"

namespace rmsmp {

// What a launch needs besides Fp6Args.
struct Fp6Patch {
  int32_t rounds;   // of step pixels until the patch is staged
  int32_t kbs;      // (tap, 32-channel block)s
  int32_t entries;  // of the table: the kbs and what the last steps look up beyond them
  int32_t unit;     // 8-byte units from one staged pixel to the next
  int32_t head;     // LDS: where the 16-byte parts begin (the 8-byte parts lie before them)
  int32_t table;    // LDS: where the table begins
  int32_t KH;
  uint32_t row_bits;  // bit KW * kh for every filter row kh
};

// What the reads of the input need, as leading scalar arguments, which the hardware hands over in registers (see
// patch_wide.h: WideFirst).
#define FP6_PATCH_FIRST_PARAMS                                                                                                       \
  const void *f_X, uint32_t f_x_bytes, int f_gx, int f_gy, uint32_t f_magic_hw, uint32_t f_magic_ow, uint32_t f_shifts, uint32_t f_w, \
      uint32_t f_h, int f_ohw, int f_ld, uint32_t f_cb
struct PatchFirst {
  const void* X;
  uint32_t x_bytes, magic_hw, magic_ow;
  int gx, gy, shift_hw, shift_ow, by_cb, W, OW, H, stride, pad, OHW, ld, CB;
  int step;  // input pixels a work-group stages at a time, CB threads each
};
#define FP6_PATCH_FIRST_UNPACK()                                                                                                        \
  PatchFirst {                                                                                                                          \
    f_X, f_x_bytes, f_magic_hw, f_magic_ow, f_gx, f_gy, (int)(f_shifts & 0xffu), (int)((f_shifts >> 8) & 0xffu), (int)(f_shifts >> 16), \
        (int)(f_w & 0xffffu), (int)(f_w >> 16), (int)(f_h & 0xffffu), (int)((f_h >> 16) & 0xffu), (int)(f_h >> 24), f_ohw, f_ld, (int)(f_cb & 0xffffu), (int)(f_cb >> 16) \
  }
#define FP6_PATCH_FIRST_ARGS(f)                                                                                                            \
  (f).X, (f).x_bytes, (f).gx, (f).gy, (f).magic_hw, (f).magic_ow, (uint32_t)((f).shift_hw | ((f).shift_ow << 8)) | ((uint32_t)(f).by_cb << 16), \
      (uint32_t)(f).W | ((uint32_t)(f).OW << 16), (uint32_t)(f).H | ((uint32_t)(f).stride << 16) | ((uint32_t)(f).pad << 24), (f).OHW, (f).ld, (uint32_t)(f).CB | ((uint32_t)(f).step << 16)

// n / d for 0 <= n < 2^31 as (2 n * magic) >> (32 + shift): without the case of d == 1, a branch
__device__ __forceinline__ int patch_div(int n, uint32_t magic, int shift) { return (int)(__umulhi((uint32_t)n * 2u, magic) >> shift); }

// What one work-group covers: 64 WM rows x 32 TN WN columns, its K steps dealt out to KS waves each.
template <int TN, int KS, int WM, int WN>
struct PatchShape {
  static constexpr int NW = KS * WM * WN, NT = LANES * NW, COLS = 32 * TN * WN;
  static constexpr int BATCH = 5;  // 16-byte pieces a thread has in flight
  static constexpr int BLOCKS = 2 * TN, OWN = BLOCKS / KS;  // 32 x 32 blocks of a wave's pair of tiles; those it finishes
  static constexpr int XCH = KS == 1 ? 0 : NW * (BLOCKS - OWN) * 16 * LANES * 4;
  // LDS: row data, the columns' pixels, then the patch
  static constexpr int PIXELS = NW * FP6_META_BYTES, PART8 = PIXELS + COLS * 8;
  static_assert(KS == 1 || OWN <= TN, "a wave finishes blocks of one tile");
};

__device__ __forceinline__ void patch_put(uint8_t* part8, uint8_t* part16, int at8, const uint4& x) {
  uint32_t lo[3], hi[3];
  fp6_widen(x.x, x.y, lo);
  fp6_widen(x.z, x.w, hi);
  *(v4i*)(part16 + 2 * at8) = (v4i){(int)lo[0], (int)lo[1], (int)lo[2], (int)hi[0]};
  *(v2i*)(part8 + at8) = (v2i){(int)hi[1], (int)hi[2]};
}

template <int I, int N, class F>
__device__ __forceinline__ void patch_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    patch_for<I + 1, N>(f);
  }
}

// A thread's pieces of the patch: block cb of every step-th pixel from q on.
struct PatchRead {
  int f_lo;        // flattened index of the first staged pixel
  uint32_t off;    // byte offset of the next piece; past the tensor for threads beyond the step * CB that have some
  uint32_t pitch;  // from there to the one after it
  int cb, q;
};

// Everything up to a wave's sums.  TWO0, TWO1: the first, the second tile has hi and lo parts (fp6_pair_joined).  SLOTS: its tiles,
// one where an odd number of them leaves one over.
template <class S, int TN, int KS, int WM, int WN, bool RAGGED, int SLOTS, bool TWO0, bool TWO1>
__device__ __forceinline__ float patch_wave(const Fp6Args& a, const Fp6Patch& g, const PatchFirst& f, uint8_t* smem, v16f (&acc)[2][TN], const Fp6Pair& pair, int n0, PatchRead& rd,
                                            __amdgpu_buffer_rsrc_t xr, uint4 (&raw)[S::BATCH], bool live) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kq = wave % KS, wn = wave / KS % WN;
  float* const meta = (float*)smem + wave * (FM_FIELDS * 64);
  uint2* const pixels = (uint2*)(smem + S::PIXELS);
  uint8_t* const part8 = smem + S::PART8;
  uint8_t* const part16 = smem + g.head;
  uint2* const table = (uint2*)(smem + g.table);

  // ---- the first reads: the patch's first batch is on its way
  const int4 row = fp6_read_meta(a, pair, lane);
  constexpr int NA0 = TWO0 ? 2 : 1, NA = SLOTS == 1 ? NA0 : NA0 + (TWO1 ? 2 : 1);  // operands a K step, of the first tile and in all
  // K steps of weights, and of activations, in flight
  constexpr int R = TN == 4 ? (NA == 4 ? 2 : NA == 3 ? 3 : 4) : NA <= 2 ? 6 : 4, D = TN == 4 ? 1 : 2;
  Fp6Frag ring[R][NA];
  const int total = (g.kbs + 1) >> 1;
  const int mine = live ? (total - kq + KS - 1) / KS : 0;  // K steps of this wave: kq, kq + KS, ..
  constexpr int STRIDE0 = NA0 * FP6_FRAG, STRIDE1 = (NA > NA0 ? NA - NA0 : 1) * FP6_FRAG;
  const __amdgpu_buffer_rsrc_t w0 = fp6_rsrc(a.w + pair.off0, (uint32_t)a.nsteps * STRIDE0);
  const __amdgpu_buffer_rsrc_t w1 = fp6_rsrc(a.w + pair.off1, (uint32_t)a.nsteps * STRIDE1);
  auto load_part = [&](int s, Fp6Frag (&f)[NA], auto part_tag) {  // parts 0 .. 2 NA - 1
    constexpr int part = decltype(part_tag)::value, i = part / 2;
    constexpr bool second = i >= NA0;
    int step = kq + KS * s;
    step = step < total ? step : total - 1;  // past the end: any valid step
    const int soff = second ? step * STRIDE1 + (i - NA0) * FP6_FRAG : step * STRIDE0 + i * FP6_FRAG;
    if constexpr (part % 2 == 0) {
      const fp6_v4u q = __builtin_amdgcn_raw_buffer_load_b128(second ? w1 : w0, lane * 16, soff, 0);
      f[i].a = (v4i){(int)q.x, (int)q.y, (int)q.z, (int)q.w};
    } else {
      const fp6_v2u d = __builtin_amdgcn_raw_buffer_load_b64(second ? w1 : w0, lane * 8 + 1024, soff, 0);
      f[i].b = (v2i){(int)d.x, (int)d.y};
    }
  };
  // (in the order in which the loop goes on: its waits count the reads issued after the one they wait for, on every way into it)
  patch_for<0, R - 1>([&](auto u) {
    patch_for<0, 2 * NA>([&](auto part) {
      load_part(decltype(u)::value, ring[decltype(u)::value], part);
      __builtin_amdgcn_sched_barrier(0);
    });
  });

  // ---- while those are in flight: accumulators; the table of (tap, block)s; every column's pixel and the taps of it that lie
  // inside the image
#pragma unroll
  for (int i = 0; i < SLOTS; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
#pragma unroll 1
  for (int c = tid; c < S::COLS; c += S::NT) {
    const int n = n0 + c;
    const int b = patch_div(n, f.magic_hw, f.shift_hw), rem = n - b * f.OHW;
    const int oh = patch_div(rem, f.magic_ow, f.shift_ow), ow = rem - oh * f.OW;
    const int ih0 = oh * f.stride - f.pad, iw0 = ow * f.stride - f.pad;
    const int kw_lo = max(0, -iw0), kw_hi = min(a.KW, f.W - iw0), kh_lo = max(0, -ih0) * a.KW, kh_hi = min(g.KH, f.H - ih0) * a.KW;
    // (bits kw_lo .. kw_hi - 1 of a filter row, and the rows kh_lo .. kh_hi - 1; at most 31 taps)
    const uint32_t cols = kw_hi > kw_lo ? (1u << kw_hi) - (1u << kw_lo) : 0u;
    const uint32_t rows = kh_hi > kh_lo ? g.row_bits & ((1u << kh_hi) - (1u << kh_lo)) : 0u;
    pixels[c] = make_uint2((uint32_t)(8 * (1 + ((b * f.H + ih0) * f.W + iw0 - rd.f_lo) * g.unit)), n < a.N ? cols * rows : 0u);
  }
#pragma unroll 1
  for (int kb = tid; kb < g.entries; kb += S::NT) {
    const int tap = fp6_div(kb, a.by_cb), cb = kb - tap * f.CB;
    const int kh = fp6_div(tap, a.by_kw), kw = tap - kh * a.KW;
    table[kb] = kb < g.kbs ? make_uint2((uint32_t)(8 * ((kh * f.W + kw) * g.unit + cb)), (uint32_t)tap) : make_uint2(0u, 31u);
  }
  if (tid == 0) {  // the block of zero points
    const uint32_t z = 0x11111111u * (uint32_t)a.zp;
    patch_put(part8, part16, 0, make_uint4(z, z, z, z));
  }
  __builtin_amdgcn_sched_barrier(0);

  // ---- the patch goes to LDS, batch by batch
  int at8 = 8 * (1 + rd.q * g.unit + rd.cb);
  const int pitch8 = 8 * f.step * g.unit;
  const bool have = rd.q < f.step;
#pragma unroll 1
  for (int round = 0;;) {
    if (have) {
#pragma unroll
      for (int u = 0; u < S::BATCH; ++u)
        if (round + u < g.rounds) patch_put(part8, part16, at8 + u * pitch8, raw[u]);
    }
    round += S::BATCH;
    if (round >= g.rounds) break;
    at8 += S::BATCH * pitch8;
#pragma unroll
    for (int u = 0; u < S::BATCH; ++u) {
      raw[u] = fp6_read_x<RAGGED>(xr, rd.off, f.x_bytes);
      rd.off += rd.pitch;
    }
  }
  const float bias = fp6_stage_meta(a, pair, row, meta, lane);
  __builtin_amdgcn_sched_barrier(0);
  fp6_barrier();

  // ---- K loop.  A step multiplies one column block after the other and reads each block's operand of D steps later as
  // soon as it is used; a step's table entry is read a step ahead of that, and the weights of R - 1 steps later arrive in the
  // registers of the step before.  A wave issues in order, so what is not a multiplication is spread out between them: the address behind a block's first
  // one, the reads behind its last.
  const int half = lane >> 5;
  int at[TN];
  uint32_t inside[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const uint2 p = pixels[(wn * TN + j) * 32 + (lane & 31)];
    at[j] = (int)p.x, inside[j] = p.y;
  }
  auto entry = [&](int s) { return table[2 * (kq + KS * s) + half]; };
  Fp6Frag b[D][TN];
  auto address = [&](int j, uint2 e) { return __builtin_amdgcn_sbfe((int)inside[j], e.y, 1) & (at[j] + (int)e.x); };
  auto read_b = [&](Fp6Frag& to, int at8) {
    to.a = *(const v4i*)(part16 + 2 * at8);
    to.b = *(const v2i*)(part8 + at8);
  };
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const uint2 e = entry(d);
#pragma unroll
    for (int j = 0; j < TN; ++j) read_b(b[d][j], address(j, e));
  }
  uint2 next = entry(D);
  auto step = [&](int s, auto u_tag, auto load_tag) {
    constexpr int u = decltype(u_tag)::value;
    constexpr bool LOAD = decltype(load_tag)::value;
    const Fp6Frag (&w)[NA] = ring[u];
    Fp6Frag (&x)[TN] = b[u % D];
    const uint2 after = entry(s + D + 1);
    __builtin_amdgcn_sched_barrier(0);
    patch_for<0, TN>([&](auto j_tag) {
      constexpr int j = decltype(j_tag)::value;
      // (of each of a block's products, what is multiplied with and where it is added: the hi parts first)
      auto multiply = [&](auto i_tag) {
        constexpr int i = decltype(i_tag)::value, HI = (TWO0 ? 1 : 0) + (SLOTS == 2 && TWO1 ? 1 : 0);
        if constexpr (i < HI) {
          constexpr int slot = TWO0 ? i : 1;
          acc[slot][j] = fp6_mfma_hi(w[slot == 0 ? 0 : NA0], x[j], acc[slot][j]);
        } else {
          acc[i - HI][j] = fp6_mfma(w[i == HI ? NA0 - 1 : NA - 1], x[j], acc[i - HI][j]);
        }
      };
      multiply(std::integral_constant<int, 0>{});
      __builtin_amdgcn_sched_barrier(0);
      int at8 = address(j, next), at16 = 2 * at8;
      asm("" : "+v"(at8), "+v"(at16));
      __builtin_amdgcn_sched_barrier(0);
      patch_for<1, NA>(multiply);
      __builtin_amdgcn_sched_barrier(0);
      x[j].a = *(const v4i*)(part16 + at16);
      x[j].b = *(const v2i*)(part8 + at8);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (LOAD)
        patch_for<2 * NA * j / TN, 2 * NA*(j + 1) / TN>([&](auto part) {
          load_part(s + R - 1, ring[(u + R - 1) % R], part);
          __builtin_amdgcn_sched_barrier(0);
        });
    });
    next = after;
  };
  int s = 0;
#pragma unroll 1
  for (; s + R <= mine; s += R) patch_for<0, R>([&](auto u) { step(s + decltype(u)::value, u, std::true_type{}); });
  patch_for<0, R - 1>([&](auto u) {
    if (s + decltype(u)::value < mine) step(s + decltype(u)::value, u, std::false_type{});
  });
  return bias;
}

// ID: see code_here.  READERS: the waves that read the code when the launch starts (touch_code), none where another body of the kernel does.
template <int TN, int KS, int WM, int WN, bool RAGGED, int ID, int READERS = 8>
__device__ __forceinline__ void patch_body(const PatchFirst& f, const Fp6Args& a, const Fp6Patch& g, const int block) {
  using S = PatchShape<TN, KS, WM, WN>;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  // the row blocks of one column block, which read the same pixels, follow each other on one XCD
  const int xcd = block & 7, slot = block >> 3;
  const int by = f.gy == 1 ? 0 : slot % f.gy, bx = (f.gy == 1 ? slot : slot / f.gy) * 8 + xcd;
  if (bx >= f.gx) return;
  const int n0 = bx * S::COLS;
  PatchRead rd;
  {
    const int b = patch_div(n0, f.magic_hw, f.shift_hw), rem = n0 - b * f.OHW;
    const int oh = patch_div(rem, f.magic_ow, f.shift_ow), ow = rem - oh * f.OW;
    rd.f_lo = max(0, (b * f.H + oh * f.stride - f.pad) * f.W + ow * f.stride - f.pad);
    rd.pitch = (uint32_t)(f.step * f.ld);
    rd.q = (int)(__umul24(threadIdx.x, (uint32_t)f.by_cb) >> 15);
    rd.cb = (int)threadIdx.x - rd.q * f.CB;
    rd.off = rd.q < f.step ? (uint32_t)((rd.f_lo + rd.q) * f.ld + rd.cb * 16) : FP6_OUTSIDE;
  }
  const __amdgpu_buffer_rsrc_t xr = fp6_rsrc(f.X, f.x_bytes);
  uint4 raw[S::BATCH];
#pragma unroll
  for (int u = 0; u < S::BATCH; ++u) {
    raw[u] = fp6_read_x<RAGGED>(xr, rd.off, f.x_bytes);
    rd.off += rd.pitch;
  }
  __builtin_amdgcn_sched_barrier(0);

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned touched = 0;
  if constexpr (READERS > 0) touched = touch_kernel<ID, S::NW, READERS>();
  const int kq = wave % KS, wn = wave / KS % WN, wm = wave / (KS * WN);
  const int q = by * WM + wm;  // (past the last pair: helps to stage the patch)
  const Fp6Pair pair = fp6_pair_joined(a, q < a.pairs ? q : a.pairs - 1);
  v16f acc[2][TN];  // (what is left over of an odd number of tiles leaves the second half alone)
  float bias;
  // (every way passes the same barriers)
#define RMSMP_PATCH_WAVE(SLOTS, TWO0, TWO1) bias = patch_wave<S, TN, KS, WM, WN, RAGGED, SLOTS, TWO0, TWO1>(a, g, f, smem, acc, pair, n0, rd, xr, raw, q < a.pairs)
  if (pair.t0 >= a.n_single) {
    if (pair.t1 < 0)
      RMSMP_PATCH_WAVE(1, true, false);
    else
      RMSMP_PATCH_WAVE(2, true, true);
  } else if (pair.t1 < 0) {
    RMSMP_PATCH_WAVE(1, false, false);
  } else if (pair.t1 >= a.n_single) {
    RMSMP_PATCH_WAVE(2, false, true);
  } else {
    RMSMP_PATCH_WAVE(2, false, false);
  }
#undef RMSMP_PATCH_WAVE
  if constexpr (READERS > 0) code_touched(touched);
  float* const meta = (float*)smem + wave * (FM_FIELDS * 64);
  meta[FM_BIAS * 64 + lane] = bias;

  auto finish = [&](auto& blocks, int i, int j0) {
    constexpr int NB = sizeof(blocks) / sizeof(v16f);
    const int t = i ? pair.t1 : pair.t0;
    if (t < 0) return;
    const int rows = lane_rows(t == a.n_tiles - 1 ? a.last_rows : TILE_M, lane);
    fp6_finish<NB, false>(a, blocks, meta + i * TILE_M + 16 * (lane >> 5), nullptr, rows, t * TILE_M + 16 * (lane >> 5), n0 + (wn * TN + j0) * 32 + (lane & 31));
  };
  if constexpr (KS == 1) {
    if (q >= a.pairs) return;
    finish(acc[0], 0, 0);
    finish(acc[1], 1, 0);
  } else {
    // The partial sums of a pair's blocks: wave kq finishes blocks kq * OWN .. of the 2 TN and parks the others for their owners.
    constexpr int BLOCKS = S::BLOCKS, OWN = S::OWN;
    float* const xch = (float*)(smem + S::NW * FP6_META_BYTES) + wave / KS * (KS * (BLOCKS - OWN) * 16 * LANES);
    v16f own[OWN];
    __syncthreads();  // the exchange lies over the patch
    auto give = [&](auto kq_tag) {
      constexpr int KQ = decltype(kq_tag)::value;
      float* dst = xch + KQ * ((BLOCKS - OWN) * 16 * LANES) + lane * 4;
      int n = 0;
#pragma unroll
      for (int x = 0; x < BLOCKS; ++x) {
        if (x / OWN == KQ) {
          own[x % OWN] = acc[x / TN][x % TN];
          continue;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) *(float4*)(dst + n * (16 * LANES) + c * (4 * LANES)) = make_float4(acc[x / TN][x % TN][4 * c], acc[x / TN][x % TN][4 * c + 1], acc[x / TN][x % TN][4 * c + 2], acc[x / TN][x % TN][4 * c + 3]);
        ++n;
      }
    };
    if (kq == 0)
      give(std::integral_constant<int, 0>{});
    else if (kq == 1)
      give(std::integral_constant<int, 1>{});
    else if (KS == 4 && kq == 2)
      give(std::integral_constant<int, KS == 4 ? 2 : 0>{});
    else if (KS == 4)
      give(std::integral_constant<int, KS == 4 ? 3 : 0>{});
    __syncthreads();
#pragma unroll
    for (int o = 0; o < OWN; ++o) {
      const int x = kq * OWN + o;
#pragma unroll
      for (int d = 1; d < KS; ++d) {
        // (giver k put block x after the blocks before it that are not its own)
        const int k = (kq + d) % KS;
        const float* src = xch + k * ((BLOCKS - OWN) * 16 * LANES) + (x < k * OWN ? x : x - OWN) * (16 * LANES) + lane * 4;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float4 v = *(const float4*)(src + c * (4 * LANES));
          own[o][4 * c] += v.x, own[o][4 * c + 1] += v.y, own[o][4 * c + 2] += v.z, own[o][4 * c + 3] += v.w;
        }
      }
    }
    if (q >= a.pairs) return;
    const int x0 = kq * OWN;
    finish(own, x0 / TN, x0 % TN);
  }
}

template <int TN, int KS, int WM, int WN>
constexpr int patch_id() { return ((TN * 8 + KS) * 8 + WM) * 8 + WN; }

template <int TN, int KS, int WM, int WN, bool RAGGED>
__global__ __launch_bounds__(LANES * KS * WM * WN, 2) void fp6_patch_kernel(FP6_PATCH_FIRST_PARAMS, Fp6Args a, Fp6Patch g) {
  constexpr int ID = patch_id<TN, KS, WM, WN>() * 2 + (RAGGED ? 1 : 0);
  patch_body<TN, KS, WM, WN, RAGGED, ID>(FP6_PATCH_FIRST_UNPACK(), a, g, (int)blockIdx.x);
  code_end<ID>();
}

// Work-groups of 4 waves where the grid is small or a layer has few rows, of 8 where it has many columns and deep K: of 14 tried on 2 600 layers
// (those below), the ten that, with the other kernels, reach 0.9994 of the best of all.
// (the first three: those of two layers in one launch, too)
#define RMSMP_PATCH_PAIR_SHAPES(X) X(2, 1, 2, 2) X(2, 2, 2, 1) X(2, 4, 2, 1)
#define RMSMP_PATCH_SHAPES(X) \
  RMSMP_PATCH_PAIR_SHAPES(X) X(4, 1, 1, 4) X(2, 1, 1, 4) X(4, 2, 2, 1) X(4, 4, 1, 1) X(4, 1, 4, 1) X(4, 2, 2, 2) X(2, 2, 4, 1)

// A launch.  patch_plan: whether the layer fits a shape, and what its estimate needs; patch_complete: the rest.
struct PatchPlan {
  PatchFirst f;
  Fp6Patch g;
  size_t lds;
};
// fp6_patch_pair.hip
int patch_launch_pair(const Fp6Args& a, const PatchPlan& p, const Fp6Args& b, const PatchPlan& q, int shape, hipStream_t s);

}  // namespace rmsmp
