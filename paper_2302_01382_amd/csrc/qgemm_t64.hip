// qgemm_t64.hip -- the fast path of mpq_qgemm (qgemm_dma.hpp) instantiated for one tile size; a
// translation unit per tile size so that the sources compile side by side.
#include "qgemm_dma.hpp"

namespace mpq {

#define MPQ_GO(W4, KB, ST) launch_dma<64, 64, 2, 2, ST, W4, KB>(a.a_q, a.w_q, a.M, a.N, a.K, a.a_scale, a.w_scale, a.per_row, a.y_out, a.acc_out, a.st, a.epi, a.n_partials, a.split, a.k_per_split, a.prepare_only)
// long_k: k tiles of 256 bytes.  With one 32 x 32 matrix instruction per wave and k substep this tile
// is bound by the latency of its barrier and of the loads behind it, paid once per k tile: twice
// the k per tile halves how often.
// two_stages: for a k of two or four tiles, which three stages would pad to three or six.
int launch_dma_64(bool w4, bool long_k, bool two_stages, const DmaArgs& a) {
  if (long_k) {
    if (two_stages) return w4 ? MPQ_GO(true, 256, 2) : MPQ_GO(false, 256, 2);
    return w4 ? MPQ_GO(true, 256, 3) : MPQ_GO(false, 256, 3);
  }
  if (two_stages) return w4 ? MPQ_GO(true, 128, 2) : MPQ_GO(false, 128, 2);
  return w4 ? MPQ_GO(true, 128, 3) : MPQ_GO(false, 128, 3);
}
#undef MPQ_GO

}  // namespace mpq
