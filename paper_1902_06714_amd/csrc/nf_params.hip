// Parameters and tendencies between the device layout and the canonical order,
// through a buffer of pinned host memory that the device reads and writes.
//
// What bounds it: PCIe for the device's side, page faults and the copy for the
// host's.  One strided copy per matrix into pageable memory instead moved each
// row by itself: 784-30-10 took 409 us, 784-1024^3-10 (11.7 MB) 23 ms and
// 4096^4-10 (202 MB) 112 ms to read.  Here a wave moves 1 KiB of the canonical
// order by one instruction per lane, whatever the rows' length.
#include "nf_internal.h"

namespace nf {

// Copies canonical elements [first, first + count) between buf and the device
// layout, 16 bytes of buf per thread.
template <class T, bool TO_BUF>
__global__ void __launch_bounds__(256)
canonical_kernel(const CanonicalSegs g, T* buf, T* dev, int64_t first, int64_t count) {
  constexpr int VW = 16 / sizeof(T);
  struct alignas(16) Vec {
    T e[VW];
  };
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * VW;
  if (i >= count) return;
  int q = 0;
  while (q + 1 < g.n && first + i >= g.s[q + 1].start) ++q;
  int64_t k = first + i - g.s[q].start;
  int64_t r = k / g.s[q].cols;
  int c = (int)(k % g.s[q].cols);
  Vec v;
  if constexpr (!TO_BUF) v = *reinterpret_cast<const Vec*>(buf + i);
#pragma unroll
  for (int j = 0; j < VW; ++j) {
    if (i + j < count) {
      T* d = dev + g.s[q].off + r * g.s[q].ld + c;
      if constexpr (TO_BUF)
        v.e[j] = *d;
      else
        *d = v.e[j];
      if (++c == g.s[q].cols) {
        c = 0;
        ++r;
      }
      if (q + 1 < g.n && first + i + j + 1 >= g.s[q + 1].start) {
        ++q;
        r = 0;
        c = 0;
      }
    } else if constexpr (TO_BUF) {
      v.e[j] = T(0);
    }
  }
  if constexpr (TO_BUF) *reinterpret_cast<Vec*>(buf + i) = v;
}

template <class T>
hipError_t launch_canonical(bool to_buf, const CanonicalSegs& g, T* buf, T* dev, int64_t first,
                            int64_t count, hipStream_t s) {
  constexpr int per = 256 * (16 / (int)sizeof(T));
  const dim3 grid((unsigned)((count + per - 1) / per));
  if (to_buf) return launch_k(canonical_kernel<T, true>, grid, 256, 0, s, g, buf, dev, first, count);
  return launch_k(canonical_kernel<T, false>, grid, 256, 0, s, g, buf, dev, first, count);
}

template hipError_t launch_canonical<float>(bool, const CanonicalSegs&, float*, float*, int64_t,
                                            int64_t, hipStream_t);
template hipError_t launch_canonical<double>(bool, const CanonicalSegs&, double*, double*, int64_t,
                                             int64_t, hipStream_t);

}  // namespace nf
