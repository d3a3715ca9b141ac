// qgemm_t192.hip -- the fast path of mpq_qgemm (qgemm_dma.hpp) instantiated for one tile size; a
// translation unit per tile size so that the sources compile side by side.
#include "qgemm_dma.hpp"

namespace mpq {

#define MPQ_GO(W4) launch_dma<192, 192, 2, 3, 2, W4>(a.a_q, a.w_q, a.M, a.N, a.K, a.a_scale, a.w_scale, a.per_row, a.y_out, a.acc_out, a.st, a.epi, a.n_partials, a.split, a.k_per_split, a.prepare_only)
// (three stages, one workgroup per CU either way: 12288 x 768 x 768 16.3 us against 15.8, K = 3072 33.0 against 32.9)
int launch_dma_192(bool w4, const DmaArgs& a) { return w4 ? MPQ_GO(true) : MPQ_GO(false); }
#undef MPQ_GO

}  // namespace mpq
