// fake_quant.hip -- the quantizer of paper Sec. 3.1 Eq. 1 in its symmetric integer form:
// code = clamp(RNE(x * inv), +-qmax), Q(x) = code * scale.  Emits any of: fp32 Q(x), int8 codes,
// packed int4 codes.  HBM-bound: 4 bytes read + 4 / 1 / 0.5 bytes written per element.
//
// Arithmetic per element: clamp x to +-absmax once (this is the clip of Eq. 1 and makes the
// clamp of the code redundant: |x| <= m gives |x*inv| <= qmax(1 + 2^-24), which rounds to at
// most qmax), then t = fma(x, inv, 1.5*2^23).  The low mantissa bits of t ARE the two's
// complement code, so bytes and nibbles are cut straight from t's bit pattern.
#include "common.hpp"

namespace mpq {

struct QConst {
  float m, inv, scale;
};

__device__ __forceinline__ QConst make_qconst(float m, int bits) {
  QConst c;
  c.m = m;
  bit_constants(m, bits, c.scale, c.inv);
  return c;
}

// t = 1.5*2^23 + code (exactly); clip of Eq. 1 applied to x first
__device__ __forceinline__ float magic_t(float x, const QConst& c) {
  const float xc = __builtin_amdgcn_fmed3f(x, -c.m, c.m);
  return __builtin_fmaf(xc, c.inv, kMagic);
}
__device__ __forceinline__ float dequant_t(float t, const QConst& c) { return (t - kMagic) * c.scale; }

__device__ __forceinline__ unsigned pack_bytes(float t0, float t1, float t2, float t3) {
  const unsigned lo = __builtin_amdgcn_perm((unsigned)bits_from_f(t1), (unsigned)bits_from_f(t0), 0x0c0c0400u);
  const unsigned hi = __builtin_amdgcn_perm((unsigned)bits_from_f(t3), (unsigned)bits_from_f(t2), 0x04000c0cu);
  return lo | hi;
}
// low nibble = even column, high nibble = odd column
__device__ __forceinline__ unsigned pack_nibbles(float t0, float t1, float t2, float t3) {
  const unsigned a = (unsigned)bits_from_f(t0) & 0xFu, b = (unsigned)bits_from_f(t1) & 0xFu;
  const unsigned c = (unsigned)bits_from_f(t2) & 0xFu, d = (unsigned)bits_from_f(t3) & 0xFu;
  return a | (b << 4) | (c << 8) | (d << 12);
}

// Outputs of four consecutive elements from flat element e on.  Any of the three pointers may lie at any
// address of its element type: the stores are 16, 4 and 2 bytes wide whatever the alignment (gfx950 stores
// to any byte address; the vector types say so to the compiler).
typedef unsigned u32_any __attribute__((aligned(1)));
typedef unsigned short u16_any __attribute__((aligned(1)));

__device__ __forceinline__ void emit4(const float4 v, const QConst& k0, const QConst& k1, const QConst& k2,
                                      const QConst& k3, int64_t e, float* y, int8_t* codes, uint8_t* packed) {
  const float t0 = magic_t(v.x, k0), t1 = magic_t(v.y, k1), t2 = magic_t(v.z, k2), t3 = magic_t(v.w, k3);
  if (y) store4(y + e, make_float4(dequant_t(t0, k0), dequant_t(t1, k1), dequant_t(t2, k2), dequant_t(t3, k3)));
  if (codes) *reinterpret_cast<u32_any*>(codes + e) = pack_bytes(t0, t1, t2, t3);
  if (packed) *reinterpret_cast<u16_any*>(packed + (e >> 1)) = (unsigned short)pack_nibbles(t0, t1, t2, t3);
}
// ... with one constant set for all four
__device__ __forceinline__ void emit4(const float4 v, const QConst& c, int64_t e, float* y, int8_t* codes,
                                      uint8_t* packed) {
  emit4(v, c, c, c, c, e, y, codes, packed);
}

// One to three elements from flat element e on (the end of a tensor or row), one lane; packed: e is a
// multiple of 4 or of an even row, and there are two of them.
__device__ __forceinline__ void emit_some(const float4 v, const QConst& k0, const QConst& k1, const QConst& k2,
                                          int64_t e, int count, float* y, int8_t* codes, uint8_t* packed) {
  const float t0 = magic_t(v.x, k0), t1 = magic_t(v.y, k1), t2 = magic_t(v.z, k2);
  if (y) {
    y[e] = dequant_t(t0, k0);
    if (count > 1) y[e + 1] = dequant_t(t1, k1);
    if (count > 2) y[e + 2] = dequant_t(t2, k2);
  }
  if (codes) {
    codes[e] = (int8_t)(bits_from_f(t0) & 0xFF);
    if (count > 1) codes[e + 1] = (int8_t)(bits_from_f(t1) & 0xFF);
    if (count > 2) codes[e + 2] = (int8_t)(bits_from_f(t2) & 0xFF);
  }
  if (packed) packed[e >> 1] = (uint8_t)(pack_nibbles(t0, t1, 0.0f, 0.0f) & 0xFFu);
}
// those elements (past the last one: the first again); all are read before the first is written
__device__ __forceinline__ float4 load_some(const float* x, int count) {
  return make_float4(x[0], x[count > 1 ? 1 : 0], x[count > 2 ? 2 : 0], 0.0f);
}
__device__ __forceinline__ void emit_tail(const float* x, const QConst& c, int64_t e, int count, float* y, int8_t* codes,
                                          uint8_t* packed) {
  emit_some(load_some(x + e, count), c, c, c, e, count, y, codes, packed);
}

// ---- per tensor, flat, 128-bit loads; n4 = n / 4 vectors, tail of n % 4 scalars ------------
__global__ __launch_bounds__(kBlock) void fq_flat(const float* __restrict__ x, int64_t n,
                                                  const float* __restrict__ absmax, int bits,
                                                  float* __restrict__ y, int8_t* __restrict__ codes,
                                                  uint8_t* __restrict__ packed, float* __restrict__ step_out) {
  const QConst c = make_qconst(absmax[0], bits);
  const int64_t tid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (step_out && tid == 0) step_out[0] = c.scale;  // the step size the codes dequantize with
  const int64_t n4 = n >> 2;
  for_each_vec4_tiled(reinterpret_cast<const float4*>(x), n4,
                      [&](const float4 v, int64_t i) { emit4(v, c, i << 2, y, codes, packed); });
  // tail: at most 3 elements, pairs stay together (n even whenever packed != null)
  if (tid == 0 && (n & 3)) emit_tail(x, c, n4 << 2, (int)(n & 3), y, codes, packed);
}

// ---- per tensor, codes only, the maximum still in parts (at most kMaxParts) --------------------
// Every workgroup folds the parts for itself (a few KB out of the L2) while its first tile is on its way.
__global__ __launch_bounds__(kBlock) void fq_parts(const float* __restrict__ x, int64_t n, const float* __restrict__ part,
                                                   int parts, float* __restrict__ absmax_out, int bits,
                                                   int8_t* __restrict__ codes, float* __restrict__ step_out) {
  constexpr int64_t tile = (int64_t)kBlock * kTileVec;
  const int64_t n4 = n >> 2, ntiles = (n4 + tile - 1) / tile;
  int64_t t = blockIdx.x;
  float4 v[kTileVec];
  auto fetch = [&]() {
#pragma unroll
    for (int u = 0; u < kTileVec; ++u) {
      const int64_t i = t * tile + threadIdx.x + u * kBlock;
      if (i < n4) v[u] = load_stream(x + 4 * i);
    }
  };
  if (t < ntiles) fetch();
  float m = 0.0f;
#pragma unroll
  for (int u = 0; u < kMaxParts / kBlock; ++u) {
    const int p = threadIdx.x + u * kBlock;
    if (p < parts) m = fmaxf(m, part[p]);
  }
  m = wave_max(m);
  __shared__ float sm[kBlock / kWave];
  if ((threadIdx.x & (kWave - 1)) == 0) sm[threadIdx.x / kWave] = m;
  __syncthreads();
  const QConst c = make_qconst(fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3])), bits);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    absmax_out[0] = c.m;
    step_out[0] = c.scale;
    if (n & 3) emit_tail(x, c, n4 << 2, (int)(n & 3), nullptr, codes, nullptr);
  }
  while (t < ntiles) {
#pragma unroll
    for (int u = 0; u < kTileVec; ++u) {
      const int64_t i = t * tile + threadIdx.x + u * kBlock;
      if (i < n4) emit4(v[u], c, i << 2, nullptr, codes, nullptr);
    }
    t += gridDim.x;
    if (t < ntiles) fetch();
  }
}

// ---- per row: one wave per (row, segment of seg columns, a multiple of 4) ------------------------
constexpr int64_t kSeg = 16384;  // the longest segment

__global__ __launch_bounds__(kBlock) void fq_rows(const float* __restrict__ x, int64_t rows,
                                                  int64_t cols, int64_t nseg, int64_t seg,
                                                  const float* __restrict__ absmax, int bits,
                                                  float* __restrict__ y, int8_t* __restrict__ codes,
                                                  uint8_t* __restrict__ packed) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t item = block_index() * (kBlock / kWave) + threadIdx.x / kWave;
  if (item >= rows * nseg) return;
  const int64_t r = item / nseg, c0 = (item - r * nseg) * seg;
  const int64_t c1 = (c0 + seg < cols) ? c0 + seg : cols;
  const QConst c = make_qconst(absmax[r], bits);
  const int64_t base = r * cols;
  int64_t i = base + c0 + 4 * lane;
  const int64_t end = base + c1;
  constexpr int64_t kStep = 4 * kWave;  // columns a wave covers per load
  for (; i + 3 * kStep + 4 <= end; i += 4 * kStep) {  // four loads in flight per lane
    const float4 v0 = load_stream(x + i), v1 = load_stream(x + i + kStep), v2 = load_stream(x + i + 2 * kStep),
                 v3 = load_stream(x + i + 3 * kStep);
    emit4(v0, c, i, y, codes, packed);
    emit4(v1, c, i + kStep, y, codes, packed);
    emit4(v2, c, i + 2 * kStep, y, codes, packed);
    emit4(v3, c, i + 3 * kStep, y, codes, packed);
  }
  for (; i + 4 <= end; i += kStep) emit4(load_stream(x + i), c, i, y, codes, packed);
  // the last cols % 4 elements of the row (an even number, starting on an even one, whenever packed != null)
  if (lane == 0 && (c1 & 3)) emit_tail(x, c, end - (c1 & 3), (int)(c1 & 3), y, codes, packed);
}

// ---- per row, short rows: LPR lanes per row (4 or 16) --------------------------------------------
// A wave per row: 100000 x 16 28 us at any alignment, 16384 x 101 8.6; 4 and 16 lanes 4.2 and 4.7.
template <int LPR>
__global__ __launch_bounds__(kBlock) void fq_rows_sub(const float* __restrict__ x, int64_t rows, int64_t cols,
                                                      const float* __restrict__ absmax, int bits,
                                                      float* __restrict__ y, int8_t* __restrict__ codes,
                                                      uint8_t* __restrict__ packed) {
  const int lr = threadIdx.x % LPR;
  const int64_t r = block_index() * (kBlock / LPR) + threadIdx.x / LPR;
  if (r >= rows) return;
  const int64_t base = r * cols;
  const int last = (int)(cols & 3);
  const QConst c = make_qconst(absmax[r], bits);
#pragma unroll 2
  for (int64_t i = 4 * lr; i + 4 <= cols; i += 4 * LPR) emit4(load4(x + base + i), c, base + i, y, codes, packed);
  // the last cols % 4 elements of the row (an even number, starting on an even one, whenever packed != null)
  if (lr == LPR - 1 && last) emit_tail(x, c, base + cols - last, last, y, codes, packed);
}

// ---- per column: a lane owns 4 adjacent columns (the last lane of a row 1 to 4) ----------------
// Narrow tensors: RW rows share a wave's 64 lanes (100000 x 16 12.5 -> 5.8 us).
template <int RW>
__global__ __launch_bounds__(kBlock) void fq_cols(const float* __restrict__ x, int64_t rows,
                                                  int64_t cols, const float* __restrict__ absmax,
                                                  int bits, float* __restrict__ y,
                                                  int8_t* __restrict__ codes,
                                                  uint8_t* __restrict__ packed) {
  constexpr int L = kWave / RW;  // lanes of a row
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int64_t c = (block_index() * L + lane % L) * 4;
  if (c >= cols) return;
  const int live = c + 4 <= cols ? 4 : (int)(cols - c);
  const int64_t row_step = (int64_t)gridDim.y * (kBlock / kWave) * RW;
  const int64_t r0 = ((int64_t)blockIdx.y * (kBlock / kWave) + wave) * RW + lane / L;
  float4 m;  // loaded as one: constant by constant, each load waits for the division before it
  if (live == 4) m = load4(absmax + c);
  else m = load_some(absmax + c, live);
  const QConst k0 = make_qconst(m.x, bits), k1 = make_qconst(m.y, bits), k2 = make_qconst(m.z, bits), k3 = make_qconst(m.w, bits);
  for (int64_t r = r0; r < rows; r += row_step) {  // one wait for both kinds of lanes
    const int64_t e = r * cols + c;
    float4 v;
    if (live == 4) v = load4(x + e);
    else v = load_some(x + e, live);
    if (live == 4) emit4(v, k0, k1, k2, k3, e, y, codes, packed);
    else emit_some(v, k0, k1, k2, e, live, y, codes, packed);
  }
}

template <int RW>
static void launch_fq_cols(const float* x, int64_t rows, int64_t cols, const float* absmax, int bits, float* y,
                           int8_t* codes, uint8_t* packed, hipStream_t st) {
  constexpr int64_t width = kWave / RW * 4, pass = kBlock / kWave * RW;  // columns and rows of a workgroup
  const int64_t gx = (cols + width - 1) / width;
  int64_t gy = ((int64_t)kNumCU * 8 + gx - 1) / gx;
  // at least 8 rows per lane, 2 where that would leave CUs without a workgroup
  int64_t max_gy = (rows + pass * 8 - 1) / (pass * 8);
  if (max_gy * gx < kNumCU) {
    max_gy = (kNumCU + gx - 1) / gx;
    if (max_gy > (rows + pass * 2 - 1) / (pass * 2)) max_gy = (rows + pass * 2 - 1) / (pass * 2);
  }
  if (gy > max_gy) gy = max_gy;
  fq_cols<RW><<<wide_grid(gx, kBlock, (unsigned)gy), kBlock, 0, st>>>(x, rows, cols, absmax, bits, y, codes, packed);
}

// mpq_fake_quant with one more output: for per-tensor granularity the kernel also leaves the step
// size scale_b in step_out[0] (what mpq_scale_from_absmax would compute in a launch of its own).
int fake_quant_launch(const float* x, int64_t rows, int64_t cols, int gran, const float* absmax, int bits,
                      float* y_out, int8_t* codes_out, uint8_t* packed4_out, float* step_out, void* stream) {
  if (!x || !absmax) return MPQ_ERR_NULL;
  if (step_out && gran != MPQ_PER_TENSOR) return MPQ_ERR_GRAN;
  if (!y_out && !codes_out && !packed4_out) return MPQ_ERR_NULL;
  if (rows <= 0 || cols <= 0 || mul_overflows(rows, cols)) return MPQ_ERR_SHAPE;
  if (gran < MPQ_PER_TENSOR || gran > MPQ_PER_COL) return MPQ_ERR_GRAN;
  if (bits < 2 || bits > 8) return MPQ_ERR_BITS;
  if (packed4_out && bits > 4) return MPQ_ERR_BITS;
  if (packed4_out && (cols & 1)) return MPQ_ERR_SHAPE;
  hipStream_t st = (hipStream_t)stream;
  const int64_t n = rows * cols;
  if (gran == MPQ_PER_TENSOR) {
    fq_flat<<<flat_grid(n >> 2, kBlock * kTileVec), kBlock, 0, st>>>(x, n, absmax, bits, y_out, codes_out, packed4_out, step_out);
  } else if (gran == MPQ_PER_ROW && cols <= 32) {
    fq_rows_sub<4><<<wide_grid((rows + 63) / 64, kBlock), kBlock, 0, st>>>(x, rows, cols, absmax, bits, y_out, codes_out, packed4_out);
  } else if (gran == MPQ_PER_ROW && cols <= 256) {
    fq_rows_sub<16><<<wide_grid((rows + 15) / 16, kBlock), kBlock, 0, st>>>(x, rows, cols, absmax, bits, y_out, codes_out, packed4_out);
  } else if (gran == MPQ_PER_ROW) {
    // few long rows: cut into segments of whole trips (1024 columns) until the chip has its waves: 4 x 300001
    // 23 -> 5.4 us, 64 x 30000 24 -> 5.1
    int64_t nseg = (2048 + rows - 1) / rows;
    if (nseg > (cols + 1023) / 1024) nseg = (cols + 1023) / 1024;
    int64_t seg = ((cols + nseg - 1) / nseg + 1023) / 1024 * 1024;
    if (seg > kSeg) seg = kSeg;
    nseg = (cols + seg - 1) / seg;
    const int64_t blocks = (rows * nseg + kBlock / kWave - 1) / (kBlock / kWave);
    if (blocks > 0x7FFFFFFF) return MPQ_ERR_SHAPE;
    fq_rows<<<wide_grid(blocks, kBlock), kBlock, 0, st>>>(x, rows, cols, nseg, seg, absmax, bits, y_out, codes_out, packed4_out);
  } else {
    if ((cols + kWave * 4 - 1) / (kWave * 4) > 0x7FFFFFFF) return MPQ_ERR_SHAPE;
    if (cols <= 16) launch_fq_cols<16>(x, rows, cols, absmax, bits, y_out, codes_out, packed4_out, st);
    else if (cols <= 64) launch_fq_cols<4>(x, rows, cols, absmax, bits, y_out, codes_out, packed4_out, st);
    else if (cols <= 128) launch_fq_cols<2>(x, rows, cols, absmax, bits, y_out, codes_out, packed4_out, st);
    else launch_fq_cols<1>(x, rows, cols, absmax, bits, y_out, codes_out, packed4_out, st);
  }
  return launch_status();
}

int fake_quant_codes_from_parts(const float* x, int64_t n, const float* part, int parts, float* absmax_out, int bits,
                                int8_t* codes_out, float* step_out, hipStream_t st) {
  fq_parts<<<flat_grid(n >> 2, kBlock * kTileVec), kBlock, 0, st>>>(x, n, part, parts, absmax_out, bits, codes_out, step_out);
  return launch_status();
}

}  // namespace mpq

using namespace mpq;

extern "C" int mpq_fake_quant(const float* x, int64_t rows, int64_t cols, int gran,
                              const float* absmax, int bits, float* y_out, int8_t* codes_out,
                              uint8_t* packed4_out, void* stream) {
  return fake_quant_launch(x, rows, cols, gran, absmax, bits, y_out, codes_out, packed4_out, nullptr, stream);
}

extern "C" int mpq_fake_quant_step(const float* x, int64_t rows, int64_t cols, const float* absmax, int bits,
                                   float* y_out, int8_t* codes_out, uint8_t* packed4_out, float* step_out,
                                   void* stream) {
  if (!step_out) return MPQ_ERR_NULL;
  if (reinterpret_cast<uintptr_t>(step_out) & 3u) return MPQ_ERR_ALIGN;
  return fake_quant_launch(x, rows, cols, MPQ_PER_TENSOR, absmax, bits, y_out, codes_out, packed4_out, step_out, stream);
}
