// absmax.hip -- max calibration (paper Sec. 3.1, first step of scale estimation): m = max |x|
// per tensor, per row or per column.  HBM-bound: 4 bytes read per element, one v_max per element.
//
// Per tensor: every block writes one partial maximum to the workspace and a one-block kernel
// folds them (and the previous value when accumulating) -- thousands of atomics on ONE address
// serialise in L2 and cost ~10 us.  Per row / per column the outputs are many addresses: |x| >= 0,
// so its bit pattern orders like its value and blocks combine with an integer atomic max (exact,
// order independent) after a fill kernel cleared the output (a kernel, not a memset node, so the
// call can be captured in a HIP graph).
#include "common.hpp"

namespace mpq {

__global__ void fill_u32(unsigned* p, int64_t n, unsigned v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// flat tensor: contiguous 16 KiB tiles dealt round-robin, the last n % 4 elements one by one
// partials: float [gridDim.x]
__global__ __launch_bounds__(kBlock) void absmax_flat(const float* __restrict__ x, int64_t n,
                                                      float* __restrict__ partials) {
  float m = 0.0f;
  const int64_t n4 = n >> 2;
  for_each_vec4_tiled(reinterpret_cast<const float4*>(x), n4, [&](const float4 a, int64_t) {
    m = fmaxf(m, fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))));
  });
  const int64_t j = (n4 << 2) + threadIdx.x;
  if (blockIdx.x == 0 && j < n) m = fmaxf(m, fabsf(x[j]));
  m = wave_max(m);
  __shared__ float sm[kBlock / kWave];
  if ((threadIdx.x & (kWave - 1)) == 0) sm[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
}

__global__ __launch_bounds__(kBlock) void absmax_finish(const float* __restrict__ partials, int np,
                                                        int accumulate, float* __restrict__ out) {
  float m = 0.0f;
#pragma unroll 8
  for (int p = threadIdx.x; p < np; p += kBlock) m = fmaxf(m, partials[p]);
  m = wave_max(m);
  __shared__ float sm[kBlock / kWave];
  if ((threadIdx.x & (kWave - 1)) == 0) sm[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float b = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
    if (accumulate) b = fmaxf(b, out[0]);
    out[0] = b;
  }
}

// Up to kOneMax elements: one workgroup, one launch.  Device time, two launches against this: 16 x 16
// 3.3 / 1.6 us, 64 x 256 3.8 / 2.1, 128 x 256 3.8 / 2.3.
constexpr int64_t kOneMax = 32768;
__global__ __launch_bounds__(kOneBlock) void absmax_one(const float* __restrict__ x, int n, int accumulate,
                                                        float* __restrict__ out) {
  float m = 0.0f;
  const int n4 = n >> 2;
#pragma unroll 8
  for (int i = threadIdx.x; i < n4; i += kOneBlock) {
    const float4 a = load4(x + 4 * i);
    m = fmaxf(m, fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))));
  }
  if ((int)threadIdx.x < (n & 3)) m = fmaxf(m, fabsf(x[(n & ~3) + threadIdx.x]));
  m = wave_max(m);
  __shared__ float sm[kOneBlock / kWave];
  if ((threadIdx.x & (kWave - 1)) == 0) sm[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = accumulate ? out[0] : 0.0f;
#pragma unroll
    for (int w = 0; w < kOneBlock / kWave; ++w) t = fmaxf(t, sm[w]);
    out[0] = t;
  }
}

// per row: one wave per (row, segment of kSeg columns)
constexpr int64_t kSeg = 16384;

// DIRECT: one segment per row and no running maximum -> plain store, no clearing pass needed
template <bool DIRECT>
__global__ __launch_bounds__(kBlock) void absmax_rows(const float* __restrict__ x, int64_t rows,
                                                      int64_t cols, int64_t nseg,
                                                      unsigned* __restrict__ out) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t item = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
  if (item >= rows * nseg) return;  // whole wave leaves together
  const int64_t r = item / nseg, seg = item - r * nseg;
  const int64_t c0 = seg * kSeg;
  const int64_t c1 = (c0 + kSeg < cols) ? c0 + kSeg : cols;
  const float* row = x + r * cols;
  float m = 0.0f;
  int64_t i = c0 + 4 * lane;
  constexpr int64_t kStep = 4 * kWave;  // columns a wave covers per load
  for (; i + 3 * kStep + 4 <= c1; i += 4 * kStep) {  // four loads in flight per lane
    const float4 a = load_stream(row + i), b = load_stream(row + i + kStep), c = load_stream(row + i + 2 * kStep),
                 d = load_stream(row + i + 3 * kStep);
    m = fmaxf(m, fmaxf(fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))),
                       fmaxf(fmaxf(fabsf(b.x), fabsf(b.y)), fmaxf(fabsf(b.z), fabsf(b.w)))));
    m = fmaxf(m, fmaxf(fmaxf(fmaxf(fabsf(c.x), fabsf(c.y)), fmaxf(fabsf(c.z), fabsf(c.w))),
                       fmaxf(fmaxf(fabsf(d.x), fabsf(d.y)), fmaxf(fabsf(d.z), fabsf(d.w)))));
  }
  for (; i + 4 <= c1; i += kStep) {
    const float4 a = load_stream(row + i);
    m = fmaxf(m, fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))));
  }
  if (lane < (int)(c1 & 3)) m = fmaxf(m, fabsf(row[(c1 & ~(int64_t)3) + lane]));  // c0 is a multiple of 4
  m = wave_max(m);
  if (lane == 0) {
    if (DIRECT) out[r] = abs_key(m);
    else atomicMax(out + r, abs_key(m));
  }
}

// per row, short rows: LPR lanes per row (4 or 16) of up to 256 columns, every row's result written by its own
// lanes.  A wave per row: 16384 x 101 5.2 us, 100000 x 16 17.5; this 3.1 and 2.6.
template <int LPR>
__global__ __launch_bounds__(kBlock) void absmax_rows_sub(const float* __restrict__ x, int64_t rows, int64_t cols,
                                                          int accumulate, float* __restrict__ out) {
  const int lr = threadIdx.x % LPR;
  int64_t r = block_index() * (kBlock / LPR) + threadIdx.x / LPR;
  const bool live = r < rows;
  if (!live) r = rows - 1;  // every lane stays active for the cross-lane steps
  const float* row = x + r * cols;
  const float before = lr == 0 && accumulate ? out[r] : 0.0f;
  float m = lr < (int)(cols & 3) ? fabsf(row[(cols & ~(int64_t)3) + lr]) : 0.0f;
#pragma unroll 2
  for (int64_t i = 4 * lr; i + 4 <= cols; i += 4 * LPR) {
    const float4 a = load4(row + i);
    m = fmaxf(m, fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))));
  }
  m = fmaxf(m, dpp<kQuadSwap1>(m));
  m = fmaxf(m, dpp<kQuadSwap2>(m));
  if (LPR == 16) {
    m = fmaxf(m, dpp<kRowHalfMirror>(m));
    m = fmaxf(m, dpp<kRowMirror>(m));
  }
  if (lr == 0 && live) out[r] = fmaxf(m, before);
}

// per column: a lane owns 4 adjacent columns (the last lane of a row 1 to 4), the 16 waves of a workgroup
// take interleaved rows and meet in LDS; blockIdx.y strides over row chunks, which meet in an atomic
// maximum per column and workgroup.  Those atomics are what bounds a kernel that has one per WAVE and
// many short row chunks: 12288 x 768 took 65 us with 4-wave workgroups of 64 rows; two of these
// workgroups per CU and one atomic per column and workgroup: 10.6 (16384 x 64: 82 -> 8.7;
// 1024 x 4096: 12.2 -> 6.2).
// DIRECT: one row chunk: its maxima are the result, and the clearing launch is spared (16 x 4096 4.3 -> 2.6 us,
// 100 x 101 5.4 -> 3.3; from 200 x 1000 on several chunks are faster).
constexpr int kColWaves = 16;
constexpr int64_t kColDirect = 128;
template <bool DIRECT>
__global__ __launch_bounds__(kColWaves * kWave) void absmax_cols(const float* __restrict__ x, int64_t rows,
                                                                 int64_t cols, int accumulate,
                                                                 unsigned* __restrict__ out) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int64_t row_step = (int64_t)gridDim.y * kColWaves;
  const int64_t r_first = (int64_t)blockIdx.y * kColWaves + wave;
  const int64_t group = block_index();
  if (group * (kWave * 4) >= cols) return;  // the whole workgroup
  const int64_t c = (group * kWave + lane) * 4;
  float4 m = make_float4(0.f, 0.f, 0.f, 0.f);
  const int live = c + 4 <= cols ? 4 : c < cols ? (int)(cols - c) : 0;  // columns this lane owns
  if (cols >= 4) {
    // the last lane of a row loads the row's last four columns, so that no lane takes a path of its own
    const float* p = x + (live == 4 ? c : cols - 4);
#pragma unroll 4
    for (int64_t r = r_first; r < rows; r += row_step) {
      const float4 a = load_stream(p + r * cols);
      m.x = fmaxf(m.x, fabsf(a.x)); m.y = fmaxf(m.y, fabsf(a.y));
      m.z = fmaxf(m.z, fabsf(a.z)); m.w = fmaxf(m.w, fabsf(a.w));
    }
    if (live == 3) m = make_float4(m.y, m.z, m.w, 0.0f);
    if (live == 2) m = make_float4(m.z, m.w, 0.0f, 0.0f);
    if (live == 1) m = make_float4(m.w, 0.0f, 0.0f, 0.0f);
  } else if (live > 0) {
    for (int64_t r = r_first; r < rows; r += row_step) {
      const float* p = x + r * cols;
      m.x = fmaxf(m.x, fabsf(p[0]));
      m.y = fmaxf(m.y, fabsf(p[live > 1 ? 1 : 0]));
      m.z = fmaxf(m.z, fabsf(p[live > 2 ? 2 : 0]));
    }
  }
  __shared__ float4 sm[kColWaves][kWave];
  sm[wave][lane] = m;
  __syncthreads();
  const int64_t col = group * (kWave * 4) + threadIdx.x;
  if (threadIdx.x < kWave * 4 && col < cols) {
    float t = 0.0f;
#pragma unroll
    for (int w = 0; w < kColWaves; ++w) t = fmaxf(t, reinterpret_cast<const float*>(sm[w])[threadIdx.x]);
    if (DIRECT) out[col] = abs_key(accumulate ? fmaxf(t, f_from_bits((int)out[col])) : t);
    else atomicMax(out + col, abs_key(t));
  }
}

__global__ void scale_from_absmax_k(const float* __restrict__ absmax, int64_t count, int bits,
                                    float* __restrict__ scale_out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  float s, inv;
  bit_constants(absmax[i], bits, s, inv);
  scale_out[i] = s;
}

}  // namespace mpq

using namespace mpq;

static unsigned absmax_flat_grid(int64_t n) { return flat_grid(n >> 2, kBlock * kTileVec); }

extern "C" size_t mpq_calibrate_absmax_workspace_bytes(int64_t rows, int64_t cols, int gran) {
  if (rows <= 0 || cols <= 0 || mul_overflows(rows, cols) || gran != MPQ_PER_TENSOR) return 0;
  // (the larger of the grids of 4-element and 1-element work items)
  const unsigned a = absmax_flat_grid(rows * cols), b = flat_grid(rows * cols, kBlock * 4);
  return (size_t)(a > b ? a : b) * sizeof(float);
}

extern "C" int mpq_calibrate_absmax(const float* x, int64_t rows, int64_t cols, int gran,
                                    int accumulate, float* absmax_out, void* ws, size_t ws_bytes,
                                    void* stream) {
  if (!x || !absmax_out) return MPQ_ERR_NULL;
  if (rows <= 0 || cols <= 0 || mul_overflows(rows, cols)) return MPQ_ERR_SHAPE;
  if (gran < MPQ_PER_TENSOR || gran > MPQ_PER_COL) return MPQ_ERR_GRAN;
  if (gran == MPQ_PER_TENSOR) {
    if (!ws || ws_bytes < mpq_calibrate_absmax_workspace_bytes(rows, cols, gran)) return MPQ_ERR_WORKSPACE;
    if (!aligned16(ws)) return MPQ_ERR_ALIGN;
  }
  hipStream_t st = (hipStream_t)stream;
  unsigned* out = reinterpret_cast<unsigned*>(absmax_out);
  const int64_t nch = channels(gran, rows, cols);
  const int64_t n = rows * cols;
  const int64_t nseg = (cols + kSeg - 1) / kSeg;
  const bool direct = gran == MPQ_PER_ROW && nseg == 1 && !accumulate;
  // grid limits are part of the argument check: nothing is enqueued before they have passed
  const int64_t row_blocks = (rows * nseg + kBlock / kWave - 1) / (kBlock / kWave);
  const int64_t cols_per_block = kWave * 4;
  const int64_t col_gx = (cols + cols_per_block - 1) / cols_per_block;
  if (gran == MPQ_PER_ROW && row_blocks > 0x7FFFFFFF) return MPQ_ERR_SHAPE;
  if (gran == MPQ_PER_COL && col_gx > 0x7FFFFFFF) return MPQ_ERR_SHAPE;
  if (gran != MPQ_PER_TENSOR && (nch + 255) / 256 > 0x7FFFFFFF) return MPQ_ERR_SHAPE;
  const bool short_rows = gran == MPQ_PER_ROW && cols <= 256;
  // row chunks: one up to kColDirect rows (half of that where a running maximum spares the clearing anyway), else
  // two workgroups per CU, at least 4 rows per wave
  const int64_t max_gy = (rows + kColWaves * 4 - 1) / (kColWaves * 4);
  int64_t col_gy = ((int64_t)kNumCU * 2 + col_gx - 1) / col_gx;
  if (col_gy > max_gy) col_gy = max_gy;
  if (rows <= (accumulate ? kColDirect / 2 : kColDirect)) col_gy = 1;
  const bool cleared = gran == MPQ_PER_ROW ? !direct && !short_rows : gran == MPQ_PER_COL && col_gy > 1;
  if (!accumulate && cleared) {
    fill_u32<<<(unsigned)((nch + 255) / 256), 256, 0, st>>>(out, nch, 0u);
  }
  if (gran == MPQ_PER_TENSOR && n <= kOneMax) {
    absmax_one<<<1, kOneBlock, 0, st>>>(x, (int)n, accumulate, absmax_out);
  } else if (gran == MPQ_PER_TENSOR) {
    const unsigned g = absmax_flat_grid(n);
    float* partials = reinterpret_cast<float*>(ws);
    absmax_flat<<<g, kBlock, 0, st>>>(x, n, partials);
    absmax_finish<<<1, kBlock, 0, st>>>(partials, (int)g, accumulate, absmax_out);
  } else if (short_rows && cols <= 32) {
    absmax_rows_sub<4><<<wide_grid((rows + 63) / 64, kBlock), kBlock, 0, st>>>(x, rows, cols, accumulate, absmax_out);
  } else if (short_rows) {
    absmax_rows_sub<16><<<wide_grid((rows + 15) / 16, kBlock), kBlock, 0, st>>>(x, rows, cols, accumulate, absmax_out);
  } else if (gran == MPQ_PER_ROW) {
    const unsigned g = (unsigned)row_blocks;
    if (direct) absmax_rows<true><<<g, kBlock, 0, st>>>(x, rows, cols, nseg, out);
    else absmax_rows<false><<<g, kBlock, 0, st>>>(x, rows, cols, nseg, out);
  } else {
    const dim3 grid = wide_grid(col_gx, kColWaves * kWave, (unsigned)col_gy);
    if (col_gy == 1) absmax_cols<true><<<grid, kColWaves * kWave, 0, st>>>(x, rows, cols, accumulate, out);
    else absmax_cols<false><<<grid, kColWaves * kWave, 0, st>>>(x, rows, cols, accumulate, out);
  }
  return launch_status();
}

extern "C" int mpq_scale_from_absmax(const float* absmax, int64_t count, int bits,
                                     float* scale_out, void* stream) {
  if (!absmax || !scale_out) return MPQ_ERR_NULL;
  if (count <= 0 || count > ((int64_t)1 << 38)) return MPQ_ERR_SHAPE;
  if (bits < 2 || bits > 8) return MPQ_ERR_BITS;
  scale_from_absmax_k<<<(unsigned)((count + 255) / 256), 256, 0, (hipStream_t)stream>>>(
      absmax, count, bits, scale_out);
  return launch_status();
}
