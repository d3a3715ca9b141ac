// qgemm_t256.hip -- the fast path of mpq_qgemm (qgemm_dma.hpp) instantiated for one tile size; a
// translation unit per tile size so that the sources compile side by side.
#include "qgemm_quad.hpp"

namespace mpq {

int launch_dma_256(bool w4, const DmaArgs& a) {
  return w4 ? launch_quad<256, 256, 2, 4, 2, true>(a) : launch_quad<256, 256, 2, 4, 2, false>(a);
}

}  // namespace mpq
