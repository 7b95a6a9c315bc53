// Host side of the FP6 patch kernel (fp6_patch.h): which layers it takes and its launches.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fp6_patch.h"
#include "fp6_plan.h"

namespace rmsmp {

// us: what a launch takes besides its work-groups; per round of staged pixels and per batch of those; per operand and
// column block that a SIMD multiplies, per operand that a work-group reads; per byte of exchanged sums; per finished 32 x 32 block;
// the share of a work-group's time that a second one on its unit adds; per such block of 32-bit output, with a bias; per megabyte of 32-bit output; how
// much of a last round overlaps the one before; per block where a lane's rows are no whole 8 bytes of output; per round of
// pixels that are no multiple of 16 bytes; per product of a wave with two tiles in two parts (fewer steps of weights in flight); per megabyte of weights beyond
// 2.5, which the L2 of an XCD does not hold beside the rest.
struct PatchTime {
  float launch, round, batch, multiply, load, exchange, block, share, block32, bias, megabyte, fluid, unaligned, ragged, heavy, weights;
};
struct PatchShapeInfo {
  int tn, ks, wm, wn, xch;
  PatchTime t;
};
#define PATCH_SHAPE(TN, KS, WM, WN) TN, KS, WM, WN, PatchShape<TN, KS, WM, WN>::XCH
// Fitted to 2 600 3x3 layers of convolution stacks and blocks (16 to 960 channels, images of 7 to 80 pixels, strides 1 and 2, 1 to 64 of them, every class
// ratio, weights warm).  On 900 others the way picked, this kernel or the others as they were chosen before it, takes 1.004 times as long as the
// best one (at most 1.14), and 0.94 of the time without this kernel, 0.77 where the call takes more than 9 us.
static const PatchShapeInfo kPatchShapes[] = {
    {PATCH_SHAPE(2, 1, 2, 2), {2.99f, 0.0905f, 0.179f, 0.0167f, 0.0123f, 0.0f, 0.317f, 0.606f, 0.33f, 0.0369f, 0.0496f, 0.289f, 0.137f, 0.0227f, 0.0943f, 0.0922f}},
    {PATCH_SHAPE(2, 2, 2, 1), {2.57f, 0.0559f, 0.371f, 0.0171f, 0.0134f, 3.14e-05f, 0.259f, 0.519f, 0.0f, 0.0468f, 0.119f, 0.0267f, 0.213f, 0.0205f, 0.0f, 0.00748f}},
    {PATCH_SHAPE(2, 4, 2, 1), {1.5f, 0.0884f, 0.0692f, 0.0283f, 0.00263f, 2.52e-05f, 0.645f, 1.09f, 0.0877f, 0.062f, 0.141f, 0.0f, 0.473f, 0.0722f, 0.0193f, 0.0f}},
    {PATCH_SHAPE(4, 1, 1, 4), {2.94f, 0.0954f, 0.156f, 0.0177f, 0.00245f, 0.0f, 0.323f, 0.582f, 0.0592f, 0.0299f, 0.0675f, 0.248f, 0.0949f, 0.0176f, 0.0882f, 0.1f}},
    {PATCH_SHAPE(2, 1, 1, 4), {2.45f, 0.101f, 0.115f, 0.0176f, 0.0128f, 0.0f, 0.461f, 0.517f, 0.0426f, 0.0253f, 0.0846f, 0.0859f, 0.103f, 0.0203f, 0.0705f, 0.0435f}},
    {PATCH_SHAPE(4, 2, 2, 1), {2.92f, 0.081f, 0.165f, 0.0153f, 0.0153f, 1.87e-05f, 0.236f, 0.481f, 0.00718f, 0.0274f, 0.085f, 0.0303f, 0.201f, 0.0391f, 0.0424f, 0.167f}},
    {PATCH_SHAPE(4, 4, 1, 1), {1.64f, 0.0804f, 0.183f, 0.005f, 0.0177f, 2.76e-05f, 0.318f, 0.538f, 0.0f, 0.0393f, 0.11f, 0.0f, 0.217f, 0.0266f, 0.0f, 0.13f}},
    {PATCH_SHAPE(4, 1, 4, 1), {3.23f, 0.111f, 0.185f, 0.0172f, 0.00673f, 0.0f, 0.192f, 0.369f, 0.0655f, 0.0283f, 0.0379f, 0.337f, 0.118f, 0.024f, 0.133f, 0.138f}},
    {PATCH_SHAPE(4, 2, 2, 2), {1.5f, 0.0996f, 0.224f, 0.0149f, 0.000867f, 1.6e-05f, 0.435f, 1.2f, 0.0f, 0.0195f, 0.13f, 0.0f, 0.196f, 0.0548f, 0.0831f, 0.58f}},
    {PATCH_SHAPE(2, 2, 4, 1), {1.5f, 0.0316f, 0.156f, 0.0191f, 0.0126f, 3.71e-05f, 0.405f, 0.719f, 0.0f, 0.0398f, 0.161f, 0.0f, 0.27f, 0.215f, 0.0205f, 0.00783f}},
};
#undef PATCH_SHAPE
constexpr int PATCH_SHAPES = (int)(sizeof(kPatchShapes) / sizeof(kPatchShapes[0])), PATCH_PAIR_SHAPES = 3;

// The division of patch_div
static void patch_div_of(int64_t d, uint32_t* magic, int* shift) {
  int s = 0;
  while (((int64_t)1 << s) < d) ++s;  // 2^(s-1) < d <= 2^s
  *magic = (uint32_t)((((unsigned __int128)1 << (31 + s)) + (uint64_t)d - 1) / (uint64_t)d);
  *shift = s;
}

static bool patch_plan(const Fp6Args& a, int KH, int B, int shape, PatchPlan* out) {
  const PatchShapeInfo& s = kPatchShapes[shape];
  // the input pixel of tap (0, 0) must not move back from one output pixel to the next, row or image
  const int64_t S = a.stride, OH = a.OHW / a.OW, row_extra = S * ((int64_t)a.W - a.OW), img_extra = (int64_t)a.W * ((int64_t)a.H - S * OH);
  if (row_extra < 0 || row_extra + img_extra + S < 0 || KH * a.KW >= 32 || a.CB >= 64) return false;
  if (a.H >= 65536 || a.W >= 65536 || a.OW >= 65536 || a.stride >= 256 || a.pad >= 256 || a.N >= (1 << 30) - 65536) return false;
  const uint32_t cols = 32u * s.tn * s.wn;
  const int64_t rows_crossed = (cols + (uint32_t)a.OW - 1) / (uint32_t)a.OW + 1, imgs_crossed = (cols + (uint32_t)a.OHW - 1) / (uint32_t)a.OHW + 1;
  int64_t px = (cols - 1) * S + 1 + (int64_t)(KH - 1) * a.W + (a.KW - 1) + rows_crossed * row_extra + imgs_crossed * (img_extra > 0 ? img_extra : 0);
  if (px >= ((int64_t)1 << 20)) return false;
  const int64_t unit = a.CB | 1;  // (odd: neighbouring pixels in different banks)
  const uint32_t waves = s.ks * s.wm * s.wn;
  PatchFirst& f = out->f;
  Fp6Patch& g = out->g;
  f.step = (int)(LANES * waves / (uint32_t)a.CB);
  g.rounds = (int)(((uint32_t)px + f.step - 1) / (uint32_t)f.step);
  px = (int64_t)g.rounds * f.step;
  const int64_t units = 1 + px * unit;
  if (units * 24 > 160 * 1024) return false;
  // 32-bit offsets of pixels before, in and behind the tensor
  if (((int64_t)B * a.H * a.W + 2 * px + (int64_t)a.pad * (a.W + 1)) * (8 * unit > a.ld ? 8 * unit : a.ld) >= ((int64_t)1 << 31) - 65536) return false;
  g.kbs = KH * a.KW * a.CB;
  g.entries = (g.kbs + 1) / 2 * 2 + 2 * 4 * s.ks;
  g.unit = (int)unit;
  g.KH = KH;
  const int64_t front = (int64_t)waves * FP6_META_BYTES, part8 = front + cols * 8;
  g.head = (int)((part8 + units * 8 + 15) / 16 * 16);
  g.table = (int)(g.head + units * 16);
  const int64_t need = std::max<int64_t>(g.table + (int64_t)g.entries * 8, front + s.xch);
  if (need > 160 * 1024) return false;
  out->lds = (size_t)need;
  f.gx = (int)(((uint32_t)a.N + cols - 1) / cols);
  f.gy = ((a.n_tiles + 1) / 2 + s.wm - 1) / s.wm;
  return (int64_t)(f.gx + 7) / 8 * 8 * f.gy <= 0x7fffffff;
}
// The rest of what the kernel is told.
static void patch_complete(const Fp6Args& a, PatchPlan* p) {
  PatchFirst& f = p->f;
  p->g.row_bits = 0;
  for (int kh = 0; kh < p->g.KH; ++kh) p->g.row_bits |= 1u << (kh * a.KW);
  f.by_cb = (32768 + a.CB - 1) / a.CB;  // (exact for thread numbers below 512)
  f.X = a.X, f.x_bytes = a.x_bytes;
  patch_div_of(a.OHW, &f.magic_hw, &f.shift_hw);
  patch_div_of(a.OW, &f.magic_ow, &f.shift_ow);
  f.W = a.W, f.OW = a.OW, f.H = a.H, f.stride = a.stride, f.pad = a.pad, f.OHW = a.OHW, f.ld = a.ld, f.CB = a.CB;
}

bool fp6_patch_fits(const Fp6Args& a, int KH, int B, int shape) {
  PatchPlan p;
  return shape < PATCH_SHAPES && patch_plan(a, KH, B, shape, &p);
}

// ---------------------------------------------------------------- the choice

// Work-groups per compute unit: of the launch, as the column blocks are dealt out to the XCDs, and at a time.
static float patch_per_unit(const PatchFirst& f) { return (float)((f.gx + 7) / 8 * f.gy) / 32.0f; }
static float patch_per_cu(const PatchShapeInfo& s, size_t lds) { return s.ks * s.wm * s.wn >= 8 || lds > 80 * 1024 ? 1.0f : 2.0f; }

// What a work-group takes by itself, in us.
static float patch_group_us(const Fp6Args& a, const PatchPlan& p, const PatchShapeInfo& s, bool ragged) {
  const PatchTime& t = s.t;
  const int waves = s.ks * s.wm * s.wn, two = a.n_tiles - a.n_single;
  // operands a K step: of the heaviest wave (a tile left over of an odd number is a wave by itself), and of a row block's waves
  const int paired = two - (a.n_tiles & 1);
  const float heavy = paired <= 0 ? (a.n_tiles == 1 ? 1.0f + two : 2.0f) : paired == 1 ? 3.0f : 4.0f;
  float all = (float)(a.n_tiles + two) / (float)p.f.gy;
  // (tiles in two parts are the last ones: the heaviest row block is the last, or where that is not a whole one the one before)
  const int rows = 2 * s.wm, last = a.n_tiles - (p.f.gy - 1) * rows;
  const int heaviest = std::max(last + std::min(two, last), p.f.gy > 1 ? rows + std::max(0, std::min(rows, two - last)) : 0);
  const float cap = patch_per_cu(s, p.lds);
  all = (float)(s.wn * s.ks) * (patch_per_unit(p.f) <= cap ? (float)heaviest : 0.5f * (all + (float)heaviest));
  const int steps = (((p.g.kbs + 1) >> 1) + s.ks - 1) / s.ks;
  const float multiply = (float)(steps * s.tn) * std::max(heavy, 0.25f * all) * t.multiply * (heavy == 4.0f ? 1.0f + t.heavy : 1.0f);
  const float megabytes = (float)((int64_t)(a.n_tiles + two) * a.nsteps) * (FP6_FRAG * 1e-6f);
  const float load = (float)steps * all * t.load * (1.0f + t.weights * std::max(0.0f, megabytes - 2.5f));
  const float stage = (float)p.g.rounds * t.round * (ragged ? 1.0f + 10.0f * t.ragged : 1.0f) + whole_up((float)p.g.rounds * 0.2f) * t.batch;
  const float block = t.block + (a.out_kind <= 1 ? t.block32 : a.M % 16 != 0 ? t.unaligned : 0.0f) + (a.bias ? t.bias : 0.0f);
  const float finish = 2.0f * s.tn / s.ks * block * (waves >= 8 ? 1.3f : 1.0f);
  return stage + std::max(multiply, load) + 0.3f * std::min(multiply, load) + finish + (float)s.xch * t.exchange;
}
// us of a launch whose compute units have per_unit work-groups each.
static float patch_launch_us(float group, float per_unit, size_t lds, const PatchShapeInfo& s) {
  const float cap = patch_per_cu(s, lds);
  const float n = std::max(1.0f, whole_up(per_unit)), full = whole_down(n / cap), rest = n - full * cap;
  const float round = group * (1.0f + (cap - 1.0f) * s.t.share);
  float time = full * round + (rest > 0.0f ? group * (1.0f + (rest - 1.0f) * s.t.share) : 0.0f);
  if (per_unit > cap) time = (1.0f - s.t.fluid) * time + s.t.fluid * per_unit / cap * round;
  return s.t.launch + time;
}
// (Beyond a round of work-groups the estimate is 12 to 18 % too fast, from a round and an eighth on, so layers that the tile kernel does faster came here: 480 to 480
// channels, 32 x 28 x 28, PoT rows as int8, 46.1 us where that takes 41.5; 288 to 764, 54 x 37 x 37, stride 2, 53.9 against 42.0.  800 3x3 layers of 12 to
// 70 G products take 1.017 times as long as the best way with this, 1.029 without, where they are repeated; among other launches 1.020 and 1.036.)
bool fp6_patch_choose(const Fp6Args& a, bool ragged, int KH, int B, int* shape, float* us) {
  bool any = false;
  for (int i = 0; i < PATCH_SHAPES; ++i) {
    const PatchShapeInfo& s = kPatchShapes[i];
    PatchPlan p;
    if (!patch_plan(a, KH, B, i, &p)) continue;
    const float rounds = patch_per_unit(p.f) / patch_per_cu(s, p.lds);
    const float time = (1.0f + std::min(0.18f, std::max(0.0f, 1.2f * (rounds - 1.0f)))) * patch_launch_us(patch_group_us(a, p, s, ragged), patch_per_unit(p.f), p.lds, s) +
                       (a.out_kind <= 1 ? s.t.megabyte * (float)((double)a.M * a.N * 4e-6) : 0.0f);
    if (time < *us) *us = time, *shape = i, any = true;
  }
  return any;
}

// What a work-group of one layer of a pair takes by itself, in us: the one with the most to multiply, and the mean.  (Those of the row blocks with tiles
// in two parts meet those with fewer, and the last one's waves without a pair leave the unit to others.)  The constants are PatchTime's; latency: from a
// weight read to its use, fewer steps of weights being in flight where a wave has tiles in two parts.
struct PatchPairGroup {
  float round, batch, multiply, load, exchange, block, bias, unaligned, latency, weights;
};
struct PatchGroup {
  float alone, mean;
};
static PatchGroup patch_pair_group_us(const Fp6Args& a, const PatchPlan& p, const PatchShapeInfo& s, const PatchPairGroup& t) {
  const int waves = s.ks * s.wm * s.wn, two = a.n_tiles - a.n_single;
  // operands a K step: of the heaviest wave (a tile left over of an odd number is a wave by itself), and of a row block's waves
  const int paired = two - (a.n_tiles & 1);
  const int heavy = paired <= 0 ? (a.n_tiles == 1 ? 1 + two : 2) : paired == 1 ? 3 : 4;
  // (tiles in two parts are the last ones: the heaviest row block is the last, or where that is not a whole one the one before)
  const int rows = 2 * s.wm, last = a.n_tiles - (p.f.gy - 1) * rows;
  const int heaviest = std::max(last + std::min(two, last), p.f.gy > 1 ? rows + std::max(0, std::min(rows, two - last)) : 0);
  const float slots = (float)(p.f.gy * s.wm), operands = (float)(a.n_tiles + two);
  const float steps = (float)((((p.g.kbs + 1) >> 1) + s.ks - 1) / s.ks);
  const float outside = 1.0f + t.weights * std::max(0.0f, operands * (float)a.nsteps * (FP6_FRAG * 1e-6f) - 2.5f);
  const float in_flight = (float)(heavy <= 2 ? (s.tn == 4 ? 3 : 5) : heavy == 3 ? (s.tn == 4 ? 2 : 3) : s.tn == 4 ? 1 : 3);  // (R - 1 of patch_wave)
  const float arrive = t.latency * outside / in_flight;
  auto products = [&](float wave, float all) {
    all *= (float)(s.wn * s.ks);
    const float multiply = steps * std::max((float)s.tn * std::max(wave, 0.25f * all) * t.multiply, arrive), load = steps * all * t.load * outside;
    return std::max(multiply, load) + 0.3f * std::min(multiply, load);
  };
  const float stage = (float)p.g.rounds * t.round + whole_up((float)p.g.rounds * 0.2f) * t.batch;
  const float block = t.block + (a.out_kind > 1 && a.M % 16 != 0 ? t.unaligned : 0.0f) + (a.bias ? t.bias : 0.0f);
  const float finish = 2.0f * s.tn / s.ks * block * (waves >= 8 ? 1.3f : 1.0f) + (float)s.xch * t.exchange;
  const float idle = 1.0f - (float)((a.n_tiles + 1) / 2) / slots;
  return PatchGroup{stage + products((float)heavy, (float)heaviest) + finish, stage + products(operands / slots, operands / (float)p.f.gy) + finish * (1.0f - 0.3f * idle)};
}

// Both layers in one shape: the larger layer's work-groups, and where those leave room on the units, or else behind them, the other's.  us, by
// shape: what the launch takes besides; shares of a work-group's time, as in PatchTime: of the heaviest one, of a second one on its unit, of one more beyond
// what the units hold, two each and one each; of the other layer's, whose few products leave the rest of it standing; of the places beside the
// larger layer's work-groups, those that take one of the other's without delay; per megabyte of 32-bit output.
// Fitted to 1 800 stage heads (64 to 256 channels, 64 to 1024 rows, 1 to 64 images of 8 to 62 pixels, nine class ratios in both storages): 5 to 7 % off;
// the shape picked takes 1.006 times as long as the best of the three, 95 of 100 within 1.04 (1.017 and 1.11 with every work-group as the mean one).
struct PatchPairTime {
  float launch, alone, share, rate2, rate1, other, free, megabyte;
  PatchPairGroup group;
};
static const PatchPairTime kPatchPairs[PATCH_PAIR_SHAPES] = {
    {4.05f, 0.938f, 0.838f, 0.752f, 1.05f, 2.63f, 0.63f, 0.0932f,
     {0.0588f, 0.302f, 0.0174f, 0.0132f, 0.0f, 0.161f, 0.0227f, 0.0296f, 0.2f, 0.00231f}},
    {3.8f, 0.897f, 0.594f, 0.607f, 0.969f, 2.67f, 0.497f, 0.0883f,
     {0.0527f, 0.283f, 0.0168f, 0.014f, 9.72e-06f, 0.333f, 0.0204f, 0.0936f, 0.363f, 0.0302f}},
    {2.13f, 0.939f, 0.0f, 0.0f, 0.797f, 2.2f, 0.0f, 0.11f,
     {0.0751f, 0.304f, 0.0195f, 0.0131f, 2.45e-05f, 0.374f, 0.0265f, 0.156f, 0.193f, 0.0131f}}};
bool fp6_patch_choose_pair(const Fp6Args& a, int KHa, const Fp6Args& b, int KHb, int B, int* shape, float* us) {
  bool any = false;
  const float megabytes = (a.out_kind <= 1 ? (float)((double)a.M * a.N * 4e-6) : 0.0f) + (b.out_kind <= 1 ? (float)((double)b.M * b.N * 4e-6) : 0.0f);
  for (int i = 0; i < PATCH_PAIR_SHAPES; ++i) {
    const PatchShapeInfo& s = kPatchShapes[i];
    const PatchPairTime& t = kPatchPairs[i];
    PatchPlan p, q;
    if (!patch_plan(a, KHa, B, i, &p) || !patch_plan(b, KHb, B, i, &q)) continue;
    const PatchGroup ga = patch_pair_group_us(a, p, s, t.group), gb = patch_pair_group_us(b, q, s, t.group);
    const float na = patch_per_unit(p.f), nb = patch_per_unit(q.f), cap = patch_per_cu(s, std::max(p.lds, q.lds));
    const bool first = ga.mean >= gb.mean;
    const float large = first ? na : nb, other = first ? nb : na, mean = first ? ga.mean : gb.mean, ratio = (first ? gb.mean : ga.mean) / mean;
    const float whole = std::max(1.0f, whole_up(large));
    const float n = std::max(whole, large + t.other * std::max(0.0f, other - t.free * std::max(0.0f, cap - whole)) * ratio);
    const float time = t.launch + t.alone * std::max(ga.alone, gb.alone) +
                       ((std::min(n, cap) - 1.0f) * t.share + std::max(0.0f, n - cap) * (cap > 1.0f ? t.rate2 : t.rate1)) * mean + t.megabyte * megabytes;
    if (time < *us) *us = time, *shape = i, any = true;
  }
  return any;
}

// ---------------------------------------------------------------- launches

static DispatchRecord patch_record(DispatchKernel kernel, int shape) {
  const PatchShapeInfo& s = kPatchShapes[shape];
  return DispatchRecord{kernel, s.tn, s.ks, s.wn, s.wm};
}

template <int TN, int KS, int WM, int WN, bool RAGGED>
static int patch_launch(const Fp6Args& a, const PatchPlan& p, hipStream_t s) {
  static std::atomic<uint64_t> allowed{0};
  if (const int rc = allow_large_lds((const void*)fp6_patch_kernel<TN, KS, WM, WN, RAGGED>, allowed)) return rc;
  const int64_t blocks = (int64_t)(p.f.gx + 7) / 8 * 8 * p.f.gy;
  hipLaunchKernelGGL((fp6_patch_kernel<TN, KS, WM, WN, RAGGED>), dim3((unsigned)blocks), dim3(LANES * KS * WM * WN), p.lds, s, FP6_PATCH_FIRST_ARGS(p.f), a, p.g);
  return (int)hipGetLastError();
}

int fp6_launch_patch_pair(Fp6Args& a, int KHa, Fp6Args& b, int KHb, int B, int shape, void* stream) {
  PatchPlan p, q;
  if (!patch_plan(a, KHa, B, shape, &p) || !patch_plan(b, KHb, B, shape, &q)) return (int)hipErrorInvalidValue;
  patch_complete(a, &p), patch_complete(b, &q);
  a.pairs = (a.n_tiles + 1) / 2, b.pairs = (b.n_tiles + 1) / 2;
  last_dispatch() = patch_record(DK_LDS_RESIDENT_PAIR, shape);
  return patch_launch_pair(a, p, b, q, shape, (hipStream_t)stream);
}

int fp6_launch_patch(Fp6Args& a, bool ragged, int KH, int B, int shape, void* stream) {
  PatchPlan p;
  if (!patch_plan(a, KH, B, shape, &p)) return (int)hipErrorInvalidValue;
  patch_complete(a, &p);
  a.pairs = (a.n_tiles + 1) / 2;
  last_dispatch() = patch_record(DK_FP6_PATCH, shape);
  hipStream_t s = (hipStream_t)stream;
  int i = 0;
#define X(TN, KS, WM, WN) \
  if (shape == i++) return ragged ? patch_launch<TN, KS, WM, WN, true>(a, p, s) : patch_launch<TN, KS, WM, WN, false>(a, p, s);
  RMSMP_PATCH_SHAPES(X)
#undef X
  return (int)hipErrorInvalidValue;
}

}  // namespace rmsmp
