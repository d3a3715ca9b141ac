// qgemm_t256.hip -- the fast path of mpq_qgemm (qgemm_dma.hpp) instantiated for one tile size; a
// translation unit per tile size so that the sources compile side by side.
#include "qgemm_quad.hpp"

namespace mpq {

// 64 x 128 of the tile per wave for int8 weights (16384 x 4096 x 1024 60.0 us against 61.7 with 128 x 64); a wave with
// packed weights expands its own W operands, so that half as many of them count more (68.8 against 61.5).
int launch_dma_256(bool w4, const DmaArgs& a) {
  return w4 ? launch_quad<256, 256, 2, 4, 2, true>(a) : launch_quad<256, 256, 4, 2, 2, false>(a);
}

}  // namespace mpq
