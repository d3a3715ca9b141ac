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
// 256 when such tiles reach three CUs in four; else 192 when it covers the problem in exactly one round with next to no
// padding (the BERT-base widths: 768 = 4 x 192 gives 12288 x 768 exactly 256 tiles); else 128 when those reach three CUs
// in four, else 64 (with half of the CUs for the 128 tile, us, 128 | 64: 4096 x 512 x 512 7.1 | 5.9, 2048 x 1024 x 1024 8.6 |
// 7.2, M x N x K).  Lines drawn where operands lie in the caches move when they come from memory, as the operands of a
// run's layers do: 12288 x 3072 x 768 in 192 tiles 51 us against 59 in 256 with warm operands, 68 against 65 with cold
// ones, 100352 x 256 x 256 in 128 tiles 23 against 26 and 42 against 32; these lines hold for cold operands.
// Stages: three, the deeper prefetch, where k is long (cold, 3 | 2: 6272 x 256 x 2304 14.0 | 16.4, 12288 x 768 x 3072 39.6 |
// 43.9), two where it is short or workgroups share the CU.  With a long k and a CU each the 64 tile takes k tiles
// of 256 (1568 x 512 x 4608 11.4 | 11.7 us).
struct FastTile {
  int side, stages, kb;
};
inline FastTile fast_tile(int64_t M, int64_t N, int64_t K, int num_cu) {
  auto tiles = [&](int64_t side) { return ((M + side - 1) / side) * ((N + side - 1) / side); };
  const int64_t most = num_cu * 3 / 4, t192 = tiles(192), t128 = tiles(128);
  if (N > 128 && tiles(256) >= most) return {256, 2, 128};
  if (N % 192 == 0 && t192 <= num_cu && t192 >= most && t192 * 192 * 192 <= M * N + M * N / 32)
    return {192, K >= 1024 ? 3 : 2, 128};
  if (N > 64 && t128 >= most) return {128, K >= 2048 || (t128 <= num_cu && K > 512) ? 3 : 2, 128};
  if (K < 1024) return {64, 2, 128};
  return {64, 3, K >= 2048 && tiles(64) <= num_cu ? 256 : 128};
}

}  // namespace mpq
