// The 128 x 128 tile of the wide kernels (nf_wide.h); a file for each tile,
// so that they compile side by side.
#include "nf_wide.h"

namespace nf {

// Eight waves of 64 x 32: both sets of accumulators fit with two waves on a SIMD.
// 784-1024^3-10, inference of 10000 (training step of 4096): one set, four waves of
// 64 x 64 345 us (479), error against fp64 3.05e-7 where the fp32 instruction
// had 2.93e-7; two sets, four waves 400 us (516), 1.1e-7; two sets, eight waves
// 3 us (18 us) less than that on one card, the same sums.
hipError_t launch_wide128(int epi, bool av, const GemmGroupT<float>& g, const int* nsplit,
                          hipStream_t s) {
  return wide_dispatch<128, 128, 64, 32, WIDE_AHEAD>(epi, av, g, nsplit, s);
}

}  // namespace nf
