// Launches of the FP6 tile kernel with neighbouring tiles joined in a wave (fp6_gemm.h: fp6_joined_kernel).
#include <hip/hip_runtime.h>

#include "fp6_gemm.h"
#include "fp6_plan.h"

namespace rmsmp {

template <int TN, int WM, int WN, bool CONV, bool RAGGED>
static int joined_launch(Fp6Args& a, hipStream_t s) {
  static std::atomic<uint64_t> allowed{0};
  if (const int rc = allow_large_lds((const void*)fp6_joined_kernel<TN, WM, WN, CONV, RAGGED>, allowed)) return rc;
  a.pairs = (a.n_tiles + 1) / 2;
  const int64_t blocks = fp6_grid(a, TN * WN, WM);
  if (blocks > 0x7fffffff) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL((fp6_joined_kernel<TN, WM, WN, CONV, RAGGED>), dim3((unsigned)blocks), dim3(LANES * WM * WN), (fp6_lds<TN, WM, WN>()), s, a);
  return (int)hipGetLastError();
}
template <int TN, int WM, int WN>
static int joined_launch_any(Fp6Args& a, bool conv, bool ragged, hipStream_t s) {
  if (conv) return ragged ? joined_launch<TN, WM, WN, true, true>(a, s) : joined_launch<TN, WM, WN, true, false>(a, s);
  return ragged ? joined_launch<TN, WM, WN, false, true>(a, s) : joined_launch<TN, WM, WN, false, false>(a, s);
}

int fp6_launch_joined(Fp6Args& a, bool conv, bool ragged, int shape, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  switch (shape) {
    case 0: return joined_launch_any<4, 4, 1>(a, conv, ragged, s);
    case 1: return joined_launch_any<2, 1, 4>(a, conv, ragged, s);
    case 2: return joined_launch_any<2, 4, 1>(a, conv, ragged, s);
    case 3: return joined_launch_any<4, 8, 1>(a, conv, ragged, s);
    default: return joined_launch_any<2, 2, 1>(a, conv, ragged, s);
  }
}

}  // namespace rmsmp
