"""The host-side rules for launch shapes (csrc/launch_shapes.hpp), compiled into a plain C++ program: a launch
counts its work items in x in 32 bits and its workgroups in y in 16, whatever the sizes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "launch_shapes.hpp"
using namespace mpq;
int main() {
  int bad = 0;
  // row tiles of the quantized layer for any K and alignment: every M that the argument check admits (its
  // 128-row tiles number at most kMaxGridY), next to the edges where the tile changes
  const int64_t ms[] = {1, 64, 4096, 64 * 65535 - 1, 64 * 65535, 64 * 65535 + 1, 5000000, 128 * 65535 - 1, 128 * 65535};
  const int64_t ns[] = {1, 3, 130, 4096}, ks[] = {1, 17, 147, 511, 512, 4607};
  for (int64_t M : ms)
    for (int64_t N : ns)
      for (int64_t K : ks) {
        const int ts = any_tile(M, N, K, 256);
        const int64_t gy = (M + ts - 1) / ts;
        if (gy > kMaxGridY || (ts != 64 && ts != 128)) { std::printf("tile %d for %lld x %lld x %lld\n", ts, (long long)M, (long long)N, (long long)K); bad = 1; }
      }
  const int64_t wants[] = {1, 2, 1 << 20, 1 << 21, 1 << 22, 1 << 23, 1 << 24, (int64_t)1 << 33, (int64_t)1 << 46};
  for (int threads : {64, 256, 512, 1024})
    for (int64_t w : wants) {
      const int64_t g = blocks_x(w, threads);
      if (g < 1 || g > w || g * threads > 0xFFFFFFFFll || (w * threads <= ((int64_t)1 << 31) && g != w)) { std::printf("grid %lld of %d for %lld\n", (long long)g, threads, (long long)w); bad = 1; }
    }
  // tiles of the fast kernels: the variants that exist, at any size the argument check admits ...
  for (int64_t M : {(int64_t)1, (int64_t)17, (int64_t)4096, (int64_t)100352, (int64_t)1 << 30, ((int64_t)1 << 31) - 1})
    for (int64_t N : {(int64_t)1, (int64_t)64, (int64_t)130, (int64_t)4096, (int64_t)1 << 20})
      for (int64_t K : {16, 32, 128, 1024, 1040, 2304, 4608, 133136})
        {
          const FastTile t = fast_tile(M, N, K, 256);
          const bool ok = t.side == 256                    ? t.stages == 2 && t.kb == 128
                          : t.side == 192 || t.side == 128 ? (t.stages == 2 || t.stages == 3) && t.kb == 128
                                                           : t.side == 64 && (t.stages == 3 || (t.stages == 2 && t.kb == 128));
          if (!ok) { std::printf("fast tile %d %d %d for %lld x %lld x %lld\n", t.side, t.stages, t.kb, (long long)M, (long long)N, (long long)K); bad = 1; }
        }
  // ... and the side that the sizes of the device tests (test_gpu_qgemm_tiles.py) are meant to reach
  const struct { int64_t M, N, K; int side; } sides[] = {
      {16381, 1024, 32, 256}, {16381, 1024, 1152, 256}, {32700, 1021, 32, 256}, {32700, 1021, 1152, 256}, {12288, 768, 32, 192},
      {12288, 768, 1152, 192}, {4093, 1022, 32, 128}, {4093, 1022, 1152, 128}, {1000, 512, 32, 64}, {333, 102, 1152, 64}};
  for (auto& c : sides)
    if (fast_tile(c.M, c.N, c.K, 256).side != c.side) { std::printf("side %d for %lld x %lld x %lld\n", fast_tile(c.M, c.N, c.K, 256).side, (long long)c.M, (long long)c.N, (long long)c.K); bad = 1; }
  // ... and the output tiles per workgroup: one for the sizes above but the second, several for the tall ones (W in 8 and 4 bits)
  const struct { int64_t M, N, K; int more8, more4; } chunks[] = {
      {16381, 1024, 128, 0, 0}, {32700, 1021, 128, 1, 1}, {12288, 768, 128, 0, 0}, {4093, 1022, 128, 0, 0}, {1000, 512, 128, 0, 0},
      {140001, 128, 32, 1, 1}, {140001, 101, 416, 1, 1}, {70001, 128, 2176, 1, 1}, {200001, 100, 160, 1, 1}, {140001, 61, 32, 1, 1},
      {140001, 61, 160, 1, 1}, {70001, 61, 1152, 1, 1}};
  for (auto& c : chunks)
    for (int w = 8; w >= 4; w -= 4) {
      const FastTile t = fast_tile(c.M, c.N, c.K, 256);
      const int lds = t.stages * t.side * (t.kb + t.kb * w / 8) + 2048;
      const int chunk = chunk_tiles((c.M + t.side - 1) / t.side, (c.N + t.side - 1) / t.side, 1, lds, 256);
      if (chunk < 1 || chunk > 4 || (chunk > 1) != (w == 8 ? c.more8 : c.more4)) { std::printf("chunk %d of %d tiles for %lld x %lld x %lld\n", chunk, t.side, (long long)c.M, (long long)c.N, (long long)c.K); bad = 1; }
    }
  // between half and three quarters of the CUs of 128 tiles the side depends on k; a short k has three stages where a
  // workgroup has its CU, or half of one, to itself
  const struct { int64_t M, N, K; int side, stages; } lines[] = {
      {1408, 2048, 1024, 64, 3}, {1408, 2048, 2560, 128, 3}, {1408, 2048, 3584, 128, 3}, {2944, 1024, 4096, 128, 3}, {2048, 1024, 4096, 64, 3},
      {24000, 128, 512, 64, 2}, {24000, 128, 1024, 128, 3}, {768, 1024, 512, 64, 2}, {768, 1024, 528, 64, 3}, {768, 1024, 896, 64, 3},
      {900, 1500, 512, 64, 2}, {900, 1500, 768, 64, 3}, {1408, 1664, 768, 64, 2}};
  for (auto& c : lines) {
    const FastTile t = fast_tile(c.M, c.N, c.K, 256);
    if (t.side != c.side || t.stages != c.stages) { std::printf("%d, %d stages for %lld x %lld x %lld\n", t.side, t.stages, (long long)c.M, (long long)c.N, (long long)c.K); bad = 1; }
  }
  // k tiles of 256 in the 64 tile: a long k with a CU per workgroup, a medium one that pads no half of them with two CUs
  const struct { int64_t M, N, K; int kb; } wide[] = {
      {48, 2304, 1280, 128}, {48, 2304, 1296, 128}, {48, 2304, 1440, 256}, {48, 2304, 1600, 128}, {512, 1024, 1792, 256},
      {520, 1024, 1792, 128}, {48, 2304, 2032, 256}, {768, 1024, 2032, 128}, {768, 1024, 2048, 256}, {1025, 1024, 2048, 128}};
  for (auto& c : wide)
    if (fast_tile(c.M, c.N, c.K, 256).kb != c.kb) { std::printf("k tiles of %d for %lld x %lld x %lld\n", fast_tile(c.M, c.N, c.K, 256).kb, (long long)c.M, (long long)c.N, (long long)c.K); bad = 1; }
  if (!bad) std::puts("shapes ok");
  return bad;
}
"""


def test_no_launch_is_larger_than_the_runtime_takes(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "shapes.cpp", tmp_path / "shapes"
    src.write_text(PROGRAM)
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2302_01382_amd", "csrc"),
                        str(src), "-o", str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert r.returncode == 0 and "shapes ok" in r.stdout, r.stdout
