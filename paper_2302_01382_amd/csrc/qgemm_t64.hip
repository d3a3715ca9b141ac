// qgemm_t64.hip -- the fast path of mpq_qgemm (qgemm_dma.hpp) instantiated for one tile size; a
// translation unit per tile size so that the sources compile side by side.
#include "qgemm_dma.hpp"

namespace mpq {

#define MPQ_GO(NS, W4, KB) launch_dma<64, 64, 2, 2, NS, W4, KB>(a.a_q, a.w_q, a.M, a.N, a.K, a.a_scale, a.w_scale, a.per_row, a.y_out, a.acc_out, a.st, a.epi, a.n_partials, a.split, a.k_per_split, a.prepare_only)
// What fast_tile and the split along k ask for.  k tiles of 256 bytes: with four matrix steps per wave and k substep
// this tile is bound by the latency of its barrier and of the loads behind it, paid once per k tile.
int launch_dma_64(bool w4, int stages, int kb, const DmaArgs& a) {
  if (kb == 256) return w4 ? MPQ_GO(3, true, 256) : MPQ_GO(3, false, 256);
  if (stages == 3) return w4 ? MPQ_GO(3, true, 128) : MPQ_GO(3, false, 128);
  return w4 ? MPQ_GO(2, true, 128) : MPQ_GO(2, false, 128);
}
#undef MPQ_GO

}  // namespace mpq
