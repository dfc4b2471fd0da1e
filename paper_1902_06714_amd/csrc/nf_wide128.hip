// The 128 x 128 tile of the wide kernels (nf_wide.h); a file for each tile,
// so that they compile side by side.
#include "nf_wide.h"

namespace nf {

hipError_t launch_wide128(int epi, bool av, const GemmGroupT<float>& g, const int* nsplit,
                          hipStream_t s) {
  return wide_dispatch<128, 128, 64, 64, WIDE_AHEAD>(epi, av, g, nsplit, s);
}

}  // namespace nf
