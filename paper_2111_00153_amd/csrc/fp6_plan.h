// Launchers of the FP6 kernels, one per source file.
#pragma once

namespace rmsmp {

struct Fp6Args;
struct DevicePacked;

// conv: activations are addressed as a convolution's; ragged: a column (pixel) is no multiple of 16 bytes.
// fp6_split.hip: a work-group of 4, 8 or 16 waves per 32 x 32 outputs.
int fp6_launch_split(const Fp6Args& a, bool conv, bool ragged, int waves, void* stream);

// Two convolutions (16-byte columns, no GELU) in one launch, 8 or 16 waves.
int fp6_launch_split_pair(const Fp6Args& a, const Fp6Args& b, int waves, void* stream);
// fp6_half.hip: the same on half weight tiles, a work-group of 4 or 8 waves per 16 rows x 16 nb columns, nb 1 or 2.
int fp6_launch_half(const Fp6Args& a, bool conv, bool ragged, int waves, int nb, void* stream);
int fp6_launch_half_pair(const Fp6Args& a, const Fp6Args& b, int waves, int nb, void* stream);
// fp6_joined.hip: the tile kernel with neighbouring tiles joined in a wave; shape: 256 x 128, 64 x 256, 256 x 64, 512 x 128, 128 x 64.
int fp6_launch_joined(Fp6Args& a, bool conv, bool ragged, int shape, void* stream);
// fp6_patch.hip: convolutions of several taps (the second layer of a pair: of any), the input in LDS; no GELU.
// _choose: sets *shape and *us to the fastest shape that is estimated to take less than *us, if there is one.  KH: filter rows, B: images.
bool fp6_patch_choose(const Fp6Args& a, bool ragged, int KH, int B, int* shape, float* us);
bool fp6_patch_fits(const Fp6Args& a, int KH, int B, int shape);
bool fp6_patch_choose_pair(const Fp6Args& a, int KHa, const Fp6Args& b, int KHb, int B, int* shape, float* us);
int fp6_launch_patch(Fp6Args& a, bool ragged, int KH, int B, int shape, void* stream);
int fp6_launch_patch_pair(Fp6Args& a, int KHa, Fp6Args& b, int KHb, int B, int shape, void* stream);
// i8_split.hip: the same work split on the int8 weights and int8 matrix instructions, 8 or 16 waves, 8-bit activations.
int i8_launch_split(const Fp6Args& a, const DevicePacked& w, int waves, void* stream);
// skinny.hip: 4-bit activations, K a multiple of 64, N <= 64; shape: 1..4 a work-group shape, 0 the rule's.
int skinny_launch(const Fp6Args& a, const DevicePacked& w, int shape, void* stream);

}  // namespace rmsmp
