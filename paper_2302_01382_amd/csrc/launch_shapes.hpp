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
// that the loop and not the output counts, else 64.  us, 128 against 64: 2999 x 1155 x 1021 15.2 / 17.4, 2000 x 258 x 2000
// 9.1 / 10.1, 3000 x 515 x 1200 10.9 / 12.7, 16384 x 1001 x 1000 54 / 55, 16384 x 501 x 100 (128 tiles of 128) 8.3 / 8.2, but 1200 x
// 1201 x 1200 (100) 11.8 / 10.7 and 1000 x 77 x 3000 7.0 / 6.5; many tiles of a medium k 16384 x 515 x 1000 43 / 39, from memory
// 56 / 54 (M x K x N).
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
// in four, else 64.  Lines drawn where operands lie in the caches move when they come from memory, as the operands of a
// run's layers do: 12288 x 3072 x 768 (M x N x K) in 192 tiles 51 us against 59 in 256 with warm operands, 68 against 65
// with cold ones, 100352 x 256 x 256 in 128 tiles 23 against 26 and 42 against 32; these lines hold for cold operands.
//
// Between half and three quarters of the CUs 128 tiles are too few for a short k and, where the 64 tiles would be more than two
// per CU, pay for a long one, for a medium one as well in a single column (two columns of 64 read A twice).  us, warm /
// cold, 128 | 64: 1408 x 2048 x 512 7.8 / 9.1 | 7.3 / 8.8, x 1024 9.4 / 11.4 | 9.6 / 12.3, packed 9.9 / 11.1 | 9.5 / 11.2, x 3072
// 16.3 / 21.9 | 19.7 / 24.3, packed 17.5 / 20.3 | 18.3 / 22.4; 1536 x 1920 x 2048 14.6 / 17.0 | 14.3 / 17.8, packed 14.5 / 16.2 |
// 13.4 / 16.3; 24000 x 128 x 512 8.1 / 10.4 | 8.0 / 10.7, x 1024 9.7 / 13.8 | 12.5 / 15.1; but 2048 x 1024 x 4096, two 64 tiles per
// CU, 18.0 / 23.9 | 15.9 / 21.9.
//
// Stages: three, the deeper prefetch, where k is long (cold, 3 | 2: 6272 x 256 x 2304 14.0 | 16.4, 12288 x 768 x 3072 39.6 |
// 43.9), two where it is short or workgroups share the CU.  64 tiles, warm / cold, 3 | 2: 768 x 1024 x 384 4.5 / 5.3 | 4.4 / 5.6,
// x 768 5.2 / 6.5 | 5.2 / 7.8; two per CU 900 x 1500 x 512 5.8 / 7.1 | 5.6 / 7.3, x 768 6.3 / 8.1 | 6.3 / 8.8; more 1408 x 1664 x 768
// 8.5 / 10.8 | 8.2 / 10.6.  With a long k and a CU each the 64 tile takes k tiles of 256 (768 x 1024 x 2048 7.4 / 9.4 against
// 7.3 / 10.2 us); up to a workgroup per two CUs a medium k does as well where it pads no half of one (warm / cold, 256 | 128, with
// the score: 48 x 2304 x 1440 8.6 / 10.3 | 8.9 / 11.0, 512 x 1024 x 1792 9.8 / 11.7 | 9.7 / 12.2; by kind and size a K of 1152 or 1280
// 0-7 % slower in 256, and with a CU each 900 x 1024 x 1440 6.9 / 7.9 | 6.6 / 8.6).
struct FastTile {
  int side, stages, kb;
};
inline FastTile fast_tile(int64_t M, int64_t N, int64_t K, int num_cu) {
  auto tiles = [&](int64_t side) { return ((M + side - 1) / side) * ((N + side - 1) / side); };
  const int64_t most = num_cu * 3 / 4, t192 = tiles(192), t128 = tiles(128);
  if (N > 128 && tiles(256) >= most) return {256, 2, 128};
  if (N % 192 == 0 && t192 <= num_cu && t192 >= most && t192 * 192 * 192 <= M * N + M * N / 32)
    return {192, K >= 1024 ? 3 : 2, 128};
  const int64_t t64 = tiles(64);
  const bool long_k = K >= (N <= 128 ? 1024 : 2560) && t128 >= num_cu / 2 && t64 > 2 * num_cu;
  if (N > 64 && (t128 >= most || long_k)) return {128, K >= 2048 || (t128 <= num_cu && K > 512) ? 3 : 2, 128};
  if (K < 1024) return {64, K > 512 && t64 <= 2 * num_cu ? 3 : 2, 128};
  const bool wide_k = K >= 2048 ? t64 <= num_cu : K > 1280 && (K + 127) / 128 % 2 == 0 && t64 <= num_cu / 2;
  return {64, 3, wide_k ? 256 : 128};
}

// Output tiles that a workgroup of the fast kernels works off, along M: the chip holds `slots` workgroups at a time (what
// the LDS allows per CU), so a launch costs about ceil(grid / slots) * chunk tile times; the length up to 4 that makes
// this smallest, the longer one on a tie (more tile boundaries without a drain).
inline int chunk_tiles(int64_t tm, int64_t tn, int split, int lds_bytes, int num_cu) {
  int per_cu = (160 * 1024) / lds_bytes;
  if (per_cu > 4) per_cu = 4;
  if (per_cu < 1) per_cu = 1;
  const int64_t slots = (int64_t)num_cu * per_cu;
  int chunk = 1;
  int64_t best = 0;
  for (int c = 1; c <= 4; ++c) {
    const int64_t grid = (tm + c - 1) / c * tn;
    const int64_t cost = (grid * split + slots - 1) / slots * c;
    if (c == 1 || cost <= best) { best = cost; chunk = c; }
  }
  return chunk;
}

}  // namespace mpq
