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

// Side of the output tile of qgemm_any: 128 (eight waves) once such tiles reach half of the CUs and k is long enough
// that the loop and not the output counts, else 64.  us, 128 against 64: 2999 x 1155 x 1021 15.8 / 17.7, 16384 x 1001 x 1000
// 54 / 62, 16384 x 501 x 100 (128 tiles of 128) 8.2 / 8.5, but 1200 x 1201 x 1200 (100) 12.0 / 10.8 and 1000 x 77 x 3000 6.9 /
// 6.6 (M x K x N).
// The grid's y counts the row tiles: more than kMaxGridY of 64 rows take 128 whatever the speed (the
// argument check admits what 128 can cover).
inline int any_tile(int64_t M, int64_t N, int64_t K, int num_cu) {
  if ((M + 63) / 64 > kMaxGridY) return 128;
  return K >= 256 && ((N + 127) / 128) * ((M + 127) / 128) >= num_cu / 2 ? 128 : 64;
}

// The tile of the fast kernels of mpq_qgemm: side of the square output tile, LDS stages, k bytes per stage.
//
// A tile costs its CU a fixed part (first loads, epilogue) and one per k tile of 128; a grid costs between its
// exact number of rounds and the whole rounds it starts (workgroups share CUs, and a chip that is not full
// clocks higher).  The three numbers per side, us, were fitted to 148 layers (64 <= M <= 100352, 64 <= N <= 4096,
// 64 <= K <= 4608, int8 and packed int4 weights, each timed with every tile): the side of least cost is on average
// 2.0 % slower than the best, where the thresholds this replaced (256 from 192 tiles on, 192 where it is exactly one
// round, 128 from 128 tiles on) were at 4.3 %.  us, before -> now: 4096 x 512 x 512 7.1 -> 6.0, 2048 x 1024 x 1024
// 8.8 -> 7.2, 12288 x 3072 x 768 59 -> 51, 3000 x 3000 x 512 16.3 -> 13.8 (M x N x K).
// Stages: two where the grid shares CUs or k is short, three where a workgroup has its CU to itself and k is
// long (1568 x 512 x 4608: 13.2 | 11.7), and then, with the 64 tile, k tiles of 256 (11.4); packed weights, whose k tiles are
// a quarter shorter, take two of those (16384 x 128 x 4096: 19.5 in three of 128 | 18.0).  With a short k in many
// rounds the stores of two workgroups of a CU are in each other's way once the weights are packed: three stages
// (16384 x 4096 x 128: 62 | 51; int8 55 | 60).
struct FastTile {
  int side, stages, kb;
};
inline FastTile fast_tile(int64_t M, int64_t N, int64_t K, bool w4, int num_cu) {
  struct Cost {
    int side;
    double tile, k_tile, whole;  // us per tile, us per k tile of 128, share of the rounds that counts as whole
  };
  const Cost costs[4] = {{256, 13.4, 1.34, 0.6}, {192, 7.4, 1.08, 0.9}, {128, 2.9, 0.58, 0.6}, {64, 1.1, 0.20, 0.8}};
  const int64_t kt = (K + 127) / 128;
  int side = 64;
  int64_t count = 0;
  double least = 0.0;
  for (const Cost& c : costs) {
    const int64_t n = ((M + c.side - 1) / c.side) * ((N + c.side - 1) / c.side);
    const double exact = n > num_cu ? (double)n / num_cu : 1.0, whole = (double)((n + num_cu - 1) / num_cu);
    const double cost = ((1.0 - c.whole) * exact + c.whole * whole) * (c.tile + c.k_tile * (double)kt);
    if (count == 0 || cost < least) {
      least = cost;
      side = c.side;
      count = n;
    }
  }
  if (side == 256 || side == 192) return {side, 2, 128};
  if (side == 128) {
    const bool alone = K > 2048 || (count <= num_cu && K > 512) || (w4 && count >= 6 * num_cu && K <= 512);
    return {128, alone ? 3 : 2, 128};
  }
  if (K <= 2304) return {64, 2, 128};
  if (w4) return {64, 2, 256};
  return {64, 3, count <= num_cu ? 256 : 128};
}

}  // namespace mpq
