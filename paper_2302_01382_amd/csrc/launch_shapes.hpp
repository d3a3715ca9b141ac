// launch_shapes.hpp -- host-side rules for the shape of a launch that do not need the HIP runtime, so that a
// plain C++ program can check them.
#pragma once

#include <stdint.h>

namespace mpq {

// A launch counts its work items per dimension in 32 bits and its workgroups in y and z in 16.  A kernel whose
// grid grows with the tensor takes at most blocks_x workgroups in x and the rest of the `want` in z; the
// last layer of z may hold more than are left.
constexpr int64_t kMaxGridY = 65535;
inline unsigned blocks_x(int64_t want, int threads) {
  const int64_t most = ((int64_t)1 << 31) / threads;
  return (unsigned)(want < most ? want : most);
}
inline unsigned blocks_z(int64_t want, int threads) {
  const int64_t x = blocks_x(want, threads);
  return (unsigned)((want + x - 1) / x);
}

// Side of the output tile of qgemm_any: 128 once such tiles fill the chip twice and k is long enough that the loop
// and not the output counts, else 64.  us, 128 against 64: 4000 x 2000 x 1500 33.0 / 41.0, 16384 x 1000 x 1001
// 62.6 / 74.3, but 4000 x 1000 x 1500 (256 tiles of 128) 27.0 / 23.6 and 12288 x 1000 x 200 32.9 / 20.7 (M x K x N).
// The grid's y counts the row tiles: more than kMaxGridY of 64 rows take 128 whatever the speed (the
// argument check admits what 128 can cover).
inline int any_tile(int64_t M, int64_t N, int64_t K, int num_cu) {
  if ((M + 63) / 64 > kMaxGridY) return 128;
  return K >= 512 && ((N + 127) / 128) * ((M + 127) / 128) >= 2 * num_cu ? 128 : 64;
}

}  // namespace mpq
