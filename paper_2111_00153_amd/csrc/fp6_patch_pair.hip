// Two convolutions on one input as one launch of the FP6 patch kernel (fp6_patch.h).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fp6_patch.h"

namespace rmsmp {

// The first layer's work-groups, which start first, read the code of both: up to 82 KB.
constexpr int PAIR_READERS = 12;

// Two layers on one input, the first blocks_a work-groups the first's (rmsmp_conv2d_pair).
template <int TN, int KS, int WM, int WN>
__global__ __launch_bounds__(LANES * KS * WM * WN, 2) void fp6_patch_pair_kernel(FP6_PATCH_FIRST_PARAMS, Fp6Args a, Fp6Patch g, PatchFirst first_b, Fp6Args b, Fp6Patch g_b, int blocks_a) {
  constexpr int ID = patch_id<TN, KS, WM, WN>();
  const int block = (int)blockIdx.x;
  if (block < blocks_a)
    patch_body<TN, KS, WM, WN, false, ID, PAIR_READERS>(FP6_PATCH_FIRST_UNPACK(), a, g, block);
  else
    patch_body<TN, KS, WM, WN, false, ID, 0>(first_b, b, g_b, block - blocks_a);
  code_end<ID>();
}

template <int TN, int KS, int WM, int WN>
static int launch_pair(const Fp6Args& a, const PatchPlan& p, const Fp6Args& b, const PatchPlan& q, hipStream_t s) {
  static std::atomic<uint64_t> allowed{0};
  if (const int rc = allow_large_lds((const void*)fp6_patch_pair_kernel<TN, KS, WM, WN>, allowed)) return rc;
  const int64_t blocks_a = (int64_t)(p.f.gx + 7) / 8 * 8 * p.f.gy, blocks_b = (int64_t)(q.f.gx + 7) / 8 * 8 * q.f.gy;
  if (blocks_a + blocks_b > 0x7fffffff) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL((fp6_patch_pair_kernel<TN, KS, WM, WN>), dim3((unsigned)(blocks_a + blocks_b)), dim3(LANES * KS * WM * WN), std::max(p.lds, q.lds), s, FP6_PATCH_FIRST_ARGS(p.f), a, p.g, q.f, b, q.g,
                     (int)blocks_a);
  return (int)hipGetLastError();
}

int patch_launch_pair(const Fp6Args& a, const PatchPlan& p, const Fp6Args& b, const PatchPlan& q, int shape, hipStream_t s) {
  int i = 0;
#define X(TN, KS, WM, WN) \
  if (shape == i++) return launch_pair<TN, KS, WM, WN>(a, p, b, q, s);
  RMSMP_PATCH_PAIR_SHAPES(X)
#undef X
  return (int)hipErrorInvalidValue;
}

}  // namespace rmsmp
