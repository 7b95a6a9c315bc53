// Host side of the FP6 patch kernel (fp6_patch.h): which layers it takes and its launches.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fp6_patch.h"
#include "fp6_plan.h"

namespace rmsmp {

// us: what a launch takes besides its work-groups; per round of staged pixels and per batch of those; per operand and
// column block that a SIMD multiplies, per operand that a work-group reads; per byte of exchanged sums; per finished 32 x 32 block;
// the share of a work-group's time that a second one on its unit adds; per such block with a bias; per megabyte of 32-bit output; per block where
// a lane's rows are no whole 8 bytes of output; per round of pixels that are no multiple of 16 bytes; from a weight read to its use (fewer steps of
// weights are in flight where a wave has tiles in two parts); per megabyte of weights beyond 2.5, which the L2 of an XCD does not hold beside
// the rest; the share of a work-group's time that one more adds beyond what the units hold at a time, two each and one each; how much of a
// round is waited for where it is not a whole one.
struct PatchTime {
  float launch, round, batch, multiply, load, exchange, block, share, bias, megabyte, unaligned, ragged, latency, weights, rate2, rate1, part;
};
struct PatchShapeInfo {
  int tn, ks, wm, wn, xch;
  PatchTime t;
};
#define PATCH_SHAPE(TN, KS, WM, WN) TN, KS, WM, WN, PatchShape<TN, KS, WM, WN>::XCH
// Fitted to 2 700 3x3 layers of convolution stacks and blocks (16 to 1024 channels, images of 7 to 80 pixels, strides 1 and 2, 1 to 64 of them, every class
// ratio in both storages, weights warm): a shape's estimate is 2 to 4 % off up to half a work-group per place, 4 to 8 % beyond a round of them.  (With
// one group time for all row blocks, whole last rounds and a term for tiles in two parts by themselves it was 3 to 12 % too fast beyond a
// round: 288 to 764 channels, 54 x 37 x 37, stride 2, 53.9 us where the tile kernel takes 42.0; 480 to 480, 32 x 28 x 28, 46.1 against 41.5.)
static const PatchShapeInfo kPatchShapes[] = {
    {PATCH_SHAPE(2, 1, 2, 2), {3.6f, 0.0588f, 0.302f, 0.0174f, 0.0132f, 0.0f, 0.161f, 1.01f, 0.0227f, 0.0878f, 0.0296f, 0.048f, 0.2f, 0.00231f, 1.27f, 1.49f, 0.826f}},
    {PATCH_SHAPE(2, 2, 2, 1), {3.19f, 0.0527f, 0.283f, 0.0168f, 0.014f, 9.72e-06f, 0.333f, 0.831f, 0.0204f, 0.0932f, 0.0936f, 0.043f, 0.363f, 0.0302f, 1.08f, 1.42f, 0.818f}},
    {PATCH_SHAPE(2, 4, 2, 1), {1.63f, 0.0751f, 0.304f, 0.0195f, 0.0131f, 2.45e-05f, 0.374f, 0.388f, 0.0265f, 0.107f, 0.156f, 0.123f, 0.193f, 0.0131f, 0.758f, 1.18f, 0.949f}},
    {PATCH_SHAPE(4, 1, 1, 4), {2.38f, 0.0978f, 8.21e-25f, 0.0194f, 0.0039f, 0.0f, 0.388f, 0.602f, 0.0272f, 0.0876f, 0.0414f, 0.0398f, 0.128f, 0.151f, 1.08f, 1.42f, 0.8f}},
    {PATCH_SHAPE(2, 1, 1, 4), {3.06f, 0.0823f, 0.167f, 0.0175f, 0.0133f, 0.0f, 0.295f, 0.883f, 0.0307f, 0.0845f, 0.031f, 0.0314f, 0.125f, 0.00851f, 1.08f, 1.41f, 0.725f}},
    {PATCH_SHAPE(4, 2, 2, 1), {3.57f, 0.0653f, 0.228f, 0.0175f, 0.0126f, 8.23e-06f, 0.217f, 0.94f, 0.0235f, 0.0894f, 0.113f, 0.0547f, 0.052f, 0.381f, 1.2f, 1.71f, 0.761f}},
    {PATCH_SHAPE(4, 4, 1, 1), {1.5f, 0.0732f, 0.205f, 0.0165f, 0.015f, 2.75e-05f, 0.3f, 0.957f, 0.0349f, 0.0768f, 0.0741f, 0.0649f, 0.00881f, 0.289f, 0.7f, 1.07f, 0.92f}},
    {PATCH_SHAPE(4, 1, 4, 1), {4.5f, 0.0788f, 0.0703f, 0.0188f, 0.0078f, 0.0f, 0.0857f, 1.1f, 0.0148f, 0.0818f, 0.0422f, 0.0562f, 0.0437f, 0.8f, 1.74f, 2.5f, 0.753f}},
    {PATCH_SHAPE(4, 2, 2, 2), {2.37f, 0.103f, 0.234f, 0.00729f, 0.0139f, 1.59e-05f, 0.227f, 0.437f, 0.0187f, 0.126f, 0.0918f, 0.076f, 0.233f, 0.0688f, 0.853f, 1.48f, 0.893f}},
    {PATCH_SHAPE(2, 2, 4, 1), {1.21f, 0.0925f, 0.275f, 0.0207f, 0.0127f, 3.41e-05f, 0.469f, 1.34f, 0.014f, 0.112f, 0.104f, 0.0929f, 0.372f, 0.0238f, 0.806f, 1.19f, 0.899f}},
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

// What a work-group takes by itself, in us: the one with the most to multiply, and the mean.  (Where there is more than one to a unit, those of
// the row blocks with tiles in two parts meet those with fewer, and the last one's waves without a pair leave the unit to others.)
struct PatchGroup {
  float alone, mean;
};
static PatchGroup patch_group_us(const Fp6Args& a, const PatchPlan& p, const PatchShapeInfo& s, bool ragged) {
  const PatchTime& t = s.t;
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
  const float stage = (float)p.g.rounds * t.round * (ragged ? 1.0f + 10.0f * t.ragged : 1.0f) + whole_up((float)p.g.rounds * 0.2f) * t.batch;
  const float block = t.block + (a.out_kind > 1 && a.M % 16 != 0 ? t.unaligned : 0.0f) + (a.bias ? t.bias : 0.0f);
  const float finish = 2.0f * s.tn / s.ks * block * (waves >= 8 ? 1.3f : 1.0f) + (float)s.xch * t.exchange;
  const float idle = 1.0f - (float)((a.n_tiles + 1) / 2) / slots;
  return PatchGroup{stage + products((float)heavy, (float)heaviest) + finish, stage + products(operands / slots, operands / (float)p.f.gy) + finish * (1.0f - 0.3f * idle)};
}
// us of a launch whose compute units have per_unit work-groups each.
static float patch_launch_us(const PatchGroup& group, float per_unit, size_t lds, const PatchShapeInfo& s) {
  const float cap = patch_per_cu(s, lds);
  const float n = std::max(1.0f, per_unit + s.t.part * (whole_up(per_unit) - per_unit));
  return s.t.launch + group.alone + (std::min(n, cap) - 1.0f) * s.t.share * group.mean + std::max(0.0f, n - cap) * (cap > 1.0f ? s.t.rate2 : s.t.rate1) * group.mean;
}
bool fp6_patch_choose(const Fp6Args& a, bool ragged, int KH, int B, int* shape, float* us) {
  bool any = false;
  for (int i = 0; i < PATCH_SHAPES; ++i) {
    const PatchShapeInfo& s = kPatchShapes[i];
    PatchPlan p;
    if (!patch_plan(a, KH, B, i, &p)) continue;
    const float time = patch_launch_us(patch_group_us(a, p, s, ragged), patch_per_unit(p.f), p.lds, s) + (a.out_kind <= 1 ? s.t.megabyte * (float)((double)a.M * a.N * 4e-6) : 0.0f);
    if (time < *us) *us = time, *shape = i, any = true;
  }
  return any;
}

// Both layers in one shape: the larger layer's work-groups, and where those leave room on the units, or else behind them, the other's.  us, by
// shape: what the launch takes besides; shares of a work-group's time, as in PatchTime: of the heaviest one, of a second one on its unit, of one more beyond
// what the units hold, two each and one each; of the other layer's, whose few products leave the rest of it standing; of the places beside the
// larger layer's work-groups, those that take one of the other's without delay; per megabyte of 32-bit output.
// Fitted to 1 800 stage heads (64 to 256 channels, 64 to 1024 rows, 1 to 64 images of 8 to 62 pixels, nine class ratios in both storages): 5 to 7 % off;
// the shape picked takes 1.006 times as long as the best of the three, 95 of 100 within 1.04 (1.017 and 1.11 with every work-group as the mean one).
struct PatchPairTime {
  float launch, alone, share, rate2, rate1, other, free, megabyte;
};
static const PatchPairTime kPatchPairs[PATCH_PAIR_SHAPES] = {
    {4.05f, 0.938f, 0.838f, 0.752f, 1.05f, 2.63f, 0.63f, 0.0932f}, {3.8f, 0.897f, 0.594f, 0.607f, 0.969f, 2.67f, 0.497f, 0.0883f}, {2.13f, 0.939f, 0.0f, 0.0f, 0.797f, 2.2f, 0.0f, 0.11f}};
bool fp6_patch_choose_pair(const Fp6Args& a, int KHa, const Fp6Args& b, int KHb, int B, int* shape, float* us) {
  bool any = false;
  const float megabytes = (a.out_kind <= 1 ? (float)((double)a.M * a.N * 4e-6) : 0.0f) + (b.out_kind <= 1 ? (float)((double)b.M * b.N * 4e-6) : 0.0f);
  for (int i = 0; i < PATCH_PAIR_SHAPES; ++i) {
    const PatchShapeInfo& s = kPatchShapes[i];
    const PatchPairTime& t = kPatchPairs[i];
    PatchPlan p, q;
    if (!patch_plan(a, KHa, B, i, &p) || !patch_plan(b, KHb, B, i, &q)) continue;
    const PatchGroup ga = patch_group_us(a, p, s, false), gb = patch_group_us(b, q, s, false);
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
