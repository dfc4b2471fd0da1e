// The 64 x 64 tile of the wide kernels (nf_wide.h) and their launcher; a file for each tile,
// so that they compile side by side.
#include "nf_wide.h"

namespace nf {

hipError_t launch_wide128(int epi, bool av, const GemmGroupT<float>& g, const int* nsplit, hipStream_t s);
hipError_t launch_wide256(int epi, bool av, const GemmGroupT<float>& g, const int* nsplit, hipStream_t s);

hipError_t launch_wide(int epi, int tile, bool a_vec, const GemmGroupT<float>& g, const int* nsplit,
                       hipStream_t s) {
  const bool tendency = epi == EPI_DW_SGD || epi == EPI_DW_PARTIAL;
  const bool forward = !tendency && epi != EPI_BWD && epi != EPI_BWD_PIECE;
  if (g.n < 1 || g.n > (tendency ? GEMM_GROUP_MAX : 1)) return hipErrorInvalidValue;
  for (int q = 0; q < g.n; ++q) {
    const GemmParamsT<float>& p = g.p[q];
    if (p.M <= 0 || p.N <= 0 || p.K <= 0 || nsplit[q] <= 0) return hipErrorInvalidValue;
    // offsets inside the rows of one tile, and those of its epilogue, stay
    // below the buffers' length
    const int64_t ld = p.lda > p.ldb ? p.lda : p.ldb;
    if ((int64_t)256 * (ld > p.ld0 ? ld : p.ld0) * 4 >= (int64_t)TILE_OOB ||
        (int64_t)256 * p.ldaux * 4 >= (int64_t)TILE_OOB)
      return hipErrorInvalidValue;
    if ((epi == EPI_FWD_STASH && p.ld1 != p.ld0) || (epi == EPI_BWD && p.ldaux != p.ld0) ||
        (epi == EPI_DW_SGD && p.ldw != p.ld0))
      return hipErrorInvalidValue;
    if (tendency || epi == EPI_FWD_PIECE || epi == EPI_BWD_PIECE) {
      if (p.nsub <= 0 || nsplit[q] % p.nsub != 0) return hipErrorInvalidValue;
      // A piece of a k-contiguous operand read 16 bytes at a time must start
      // on a whole stage (nf_split.h).  The tendencies split the batch,
      // which is not the contiguous index of either of their operands.
      if (!tendency && !k_pieces_aligned(nsplit[q] / p.nsub, p.shard_len, p.nsub, p.sub_len))
        return hipErrorInvalidValue;
    } else if (nsplit[q] != 1) {
      return hipErrorInvalidValue;
    }
  }
  const bool av = forward ? a_vec : true;
  if (tile == TILE_256x256) return launch_wide256(epi, av, g, nsplit, s);
  if (tile == TILE_128x128) return launch_wide128(epi, av, g, nsplit, s);
  // At most 32 k are all prologue and epilogue, in which the loading waves have
  // no part: four waves that load and multiply (tendencies of one sample, 1024 x 2000
  // 10.1 us with loading waves, 8.8 without, of 48 samples 10.8 and 10.6; inference of
  // 150 nets of five to nine layers of 8 to 200 units takes 0.98 of the time)
  int k = 0;
  for (int q = 0; q < g.n; ++q) {
    const int len = nsplit[q] > 1 ? g.p[q].sub_len : g.p[q].K;
    k = len > k ? len : k;
  }
  if (k <= 32) return wide_dispatch<64, 64, 32, 32, WIDE_PLAIN>(epi, av, g, nsplit, s);
  return wide_dispatch<64, 64, 32, 32, WIDE_ROLES>(epi, av, g, nsplit, s);
}

}  // namespace nf
