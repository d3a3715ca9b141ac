// quant_error.hip -- the sum under the expectation of paper Sec. 3.2.1 Eq. 2,
// SSE_b = sum (Q_b(x) - x)^2, for every bit-width b_lo..b_hi in ONE read of the tensor, per
// tensor / per row / per column; plus the two-tensor squared distance used as the candidate score.
//
// Per element and bit-width: t = fma(xc, inv_b, 1.5*2^23); q = t - 1.5*2^23; e = fma(q, scale_b, -x);
// acc_b = fma(e, e, acc_b) -- four VALU operations, with xc = clip(x, +-m) computed once (it
// replaces the clamp of the code, see fake_quant.hip; two bits take three, see sweep.hpp).
// 28 lane-operations per element for the full sweep b = 2..8 against 4 bytes of HBM traffic: a
// quarter below what the vector ALUs take
// from registers (mpq_diag_sweep_alu_rate), so the kernel is bound by HBM as long as nothing else
// gets into the inner loop (constants live in registers for the whole kernel, loads are 128-bit
// and four deep).
//
// Reproducibility: per-lane fp32 partial sums (a lane adds at most ~4k elements one after the other; per column
// rows * groups of 256 columns / 8192 of them, at least 8), fixed-order DPP wave reduction, then double
// precision across waves / blocks in a fixed order.  No float atomics anywhere.
#include "common.hpp"
#include "sweep.hpp"

#include <mutex>
#include <type_traits>

namespace mpq {

constexpr int64_t kSeg = 16384;  // columns per wave item in the per-row kernels

// ---- per tensor ----------------------------------------------------------------------------
// partials: double [gridDim.x][NB]
// PLAN: a tensor that a sweep plan can hold, summed as the batched kernels do (bit for bit); any other in tiles or,
// small ones, one vector a trip
template <int NB, bool PLAN, bool TILED>
__global__ __launch_bounds__(kBlock) void qe_flat(const float* __restrict__ x, int64_t n,
                                                  const float* __restrict__ absmax, int b_lo,
                                                  double* __restrict__ partials) {
  std::conditional_t<PLAN, Sweep<NB>, Sweep4<NB>> s;
  s.init(absmax[0], b_lo);
  s.clear();
  const int64_t n4 = n >> 2;
  if (TILED) for_each_vec4_tiled<PLAN>(reinterpret_cast<const float4*>(x), n4, [&](const float4 v, int64_t) { s.add4(v); });
  else for_each_vec4_strided(x, n4, [&](const float4 v) { s.add4(v); });
  const int64_t j = (n4 << 2) + threadIdx.x;  // the last n % 4 elements
  if (blockIdx.x == 0 && j < n) s.add(x[j]);
  using Sum = std::conditional_t<PLAN, float, double>;
  __shared__ Sum sm[kBlock / kWave][NB];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    Sum w;
    if constexpr (PLAN) w = wave_sum(s.total(b));
    else w = wave_sum_rows(s.total(b));
    if (lane == 0) sm[wave][b] = w;
  }
  __syncthreads();
  if (threadIdx.x < NB)
    partials[(int64_t)blockIdx.x * NB + threadIdx.x] =
        ((double)sm[0][threadIdx.x] + (double)sm[1][threadIdx.x]) +
        ((double)sm[2][threadIdx.x] + (double)sm[3][threadIdx.x]);
}

// Up to kOneLimit / NB elements and kOneMost (a quarter of it at any alignment, where two launches have chains of four
// as well): one workgroup, one launch; a lane has an fp32 sum per element of a
// vector, and double takes over from rows of sixteen lanes on.  Device time for b = 2..8, two launches against this: 64 x 64 5.7 / 4.6 us, 64 x 128
// 6.0 / 5.3, 64 x 256 6.1 / 6.2 (and a launch, 4.3 us of the host's time, less); for one width 128 x 256 4.3 / 2.8,
// 256 x 256 4.3 / 3.7, from 80000 elements on two launches are faster.
constexpr int64_t kOneLimit = 7 * 16384, kOneMost = 65536;
template <int NB>
__global__ __launch_bounds__(kOneBlock) void qe_one(const float* __restrict__ x, int n,
                                                    const float* __restrict__ absmax, int b_lo,
                                                    double* __restrict__ out) {
  constexpr int NW = kOneBlock / kWave;
  Sweep4<NB> s;
  s.init(absmax[0], b_lo);
  s.clear();
  const int n4 = n >> 2;
#pragma unroll 4
  for (int i = threadIdx.x; i < n4; i += kOneBlock) s.add4(load4(x + 4 * i));
  if ((int)threadIdx.x < (n & 3)) s.add(x[(n & ~3) + threadIdx.x]);
  __shared__ double sm[NW][NB];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const double w = wave_sum_rows(s.total(b));
    if (lane == 0) sm[wave][b] = w;
  }
  __syncthreads();
  if (threadIdx.x < NB) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += sm[w][threadIdx.x];
    out[threadIdx.x] = t;
  }
}

// out[b] = sum_p partials[p][b], p < np, in a fixed order: thread t adds p = t, t + 256, ...
// (independent loads, unrolled), then a fixed LDS tree over the 256 threads.
template <int NB>
__global__ __launch_bounds__(kBlock) void qe_finish_tree(const double* __restrict__ partials,
                                                         int64_t np, double* __restrict__ out) {
  double a[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) a[b] = 0.0;
#pragma unroll 4
  for (int64_t p = threadIdx.x; p < np; p += kBlock) {
#pragma unroll
    for (int b = 0; b < NB; ++b) a[b] += partials[p * NB + b];
  }
  __shared__ double sm[kBlock][NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) sm[threadIdx.x][b] = a[b];
  __syncthreads();
  for (int half = kBlock / 2; half >= 1; half >>= 1) {
    if ((int)threadIdx.x < half) {
#pragma unroll
      for (int b = 0; b < NB; ++b) sm[threadIdx.x][b] += sm[threadIdx.x + half][b];
    }
    __syncthreads();
  }
  if (threadIdx.x < NB) out[threadIdx.x] = sm[0][threadIdx.x];
}

// out[k] = sum_p partials[k + p * stride] (per-column kernels: planes of nch * nb sums) or, rows cut into
// segments, with the nb sums of a row's segments next to each other: k / nb * stride_ch + k % nb + p * stride.
// 64 outputs per workgroup; wave w adds the partials p = w, w + 4, ... and the four meet in a fixed order.
__global__ __launch_bounds__(kBlock) void qe_finish_planes(const double* __restrict__ partials, int64_t nch, int64_t np,
                                                           int nb, int64_t stride_ch, int64_t stride_p,
                                                           double* __restrict__ out) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  __shared__ double sm[kBlock / kWave][kWave];
  const int64_t k = block_index() * kWave + lane;
  const bool live = k < nch * nb;
  double a = 0.0;
  if (live) {
    const int64_t ch = k / nb;
    const double* src = partials + ch * stride_ch + (k - ch * nb);
#pragma unroll 8
    for (int64_t p = wave; p < np; p += kBlock / kWave) a += src[p * stride_p];
  }
  sm[wave][lane] = a;
  __syncthreads();
  if (wave == 0 && live) out[k] = (sm[0][lane] + sm[1][lane]) + (sm[2][lane] + sm[3][lane]);
}

// ---- per row, rows of several segments: one wave per (row, segment) -----------------------------
// dst: partials [rows][nseg][NB]
template <int NB>
__global__ __launch_bounds__(kBlock) void qe_rows(const float* __restrict__ x, int64_t rows,
                                                  int64_t cols, int64_t nseg,
                                                  const float* __restrict__ absmax, int b_lo,
                                                  double* __restrict__ dst) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t item = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
  if (item >= rows * nseg) return;  // the whole wave leaves together
  const int64_t r = item / nseg, seg = item - r * nseg;
  const int64_t c0 = seg * kSeg;
  const int64_t c1 = (c0 + kSeg < cols) ? c0 + kSeg : cols;
  Sweep<NB> s;
  s.init(absmax[r], b_lo);
  const float* row = x + r * cols;
  const float4* r4 = reinterpret_cast<const float4*>(row);  // 4-byte aligned: see load_stream
  int64_t i = (c0 >> 2) + lane;
  const int64_t e4 = c1 >> 2;
  for (; i + 3 * kWave < e4; i += 4 * kWave) {
    const float4 a = load_stream(r4 + i), b = load_stream(r4 + i + kWave), c = load_stream(r4 + i + 2 * kWave),
                 d = load_stream(r4 + i + 3 * kWave);
    s.add4(a); s.add4(b); s.add4(c); s.add4(d);
  }
  for (; i < e4; i += kWave) s.add4(load_stream(r4 + i));
  if (lane < (int)(c1 & 3)) s.add(row[(e4 << 2) + lane]);
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const float w = wave_sum(s.acc[b]);
    if (lane == 0) dst[item * NB + b] = (double)w;
  }
}

// ---- per row, short rows: LPR lanes per row (16 or 64), 64 / LPR rows per wave ---------------------
// The 2 NB per-row constants cost a division each; here lane j of a row group computes constant j
// only and the group shares them through the cross-lane network, and the final sums need 4 DPP
// steps instead of a full wave reduction.  cols <= kSeg.
// PLAN: a tensor that a sweep plan can hold: the sums are formed as the batched kernels form them, so that the two
// calls agree bit for bit.  Any other: rows start anywhere, so neighbouring vectors share lines, and cached loads
// beat streaming ones (16384 x 255, 16 lanes: 7.5 / 7.4 us, 300 x 1023, 64 lanes: 4.5 / 3.7, one width of 4000 x 101
// 2.9 / 2.4); and a lane has a sum per element of a vector, which keeps its fp32 chains at cols / (4 LPR).
template <int NB, int LPR, bool PLAN>
__global__ __launch_bounds__(kBlock) void qe_rows_sub(const float* __restrict__ x, int64_t rows,
                                                      int64_t cols, const float* __restrict__ absmax,
                                                      int b_lo, double* __restrict__ out) {
  constexpr int RW = kWave / LPR;  // rows per wave
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int lr = lane % LPR;
  int64_t r = ((int64_t)blockIdx.x * (kBlock / kWave) + wave) * RW + lane / LPR;
  const bool live = r < rows;
  if (!live) r = rows - 1;  // keep every lane active for the cross-lane steps; result discarded
  const float m = absmax[r];
  const float4* r4 = reinterpret_cast<const float4*>(x + r * cols);
  const int64_t e4 = cols >> 2;
  std::conditional_t<PLAN, Sweep<NB>, Sweep4<NB>> s;
  auto constants = [&]() {
    s.clear();
    s.m = m;
    // lane j < 7: inv of bit-width b_lo + j; lane 7 + j: scale of bit-width b_lo + j
    const int j = lr < 7 ? lr : lr - 7;
    float sc, inv;
    bit_constants(m, b_lo + (j < NB ? j : 0), sc, inv);
    const float mine = lr < 7 ? inv : sc;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      s.inv[b] = __shfl(mine, b, LPR);
      s.sc[b] = __shfl(mine, 7 + b, LPR);
    }
  };
  if constexpr (PLAN) {  // cols % 4 == 0
    constants();
    int64_t i = lr;
    for (; i + 3 * LPR < e4; i += 4 * LPR) {
      const float4 a = load_stream(r4 + i), b = load_stream(r4 + i + LPR), c = load_stream(r4 + i + 2 * LPR),
                   d = load_stream(r4 + i + 3 * LPR);
      s.add4(a); s.add4(b); s.add4(c); s.add4(d);
    }
    for (; i < e4; i += LPR) s.add4(load_stream(r4 + i));
  } else {
    // four vectors in flight per lane, the first ones in front of the constants, those that are left at the
    // end of a row as well; vectors past the row's end are zeros, which add nothing
    auto load = [&](int64_t i) { return load4(reinterpret_cast<const float*>(r4 + i)); };
    auto fetch = [&](float4 (&v)[4], int64_t i0) {
      if (i0 + 4 * LPR <= e4) {  // the same for all lanes of the wave
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = load(i0 + k * LPR + lr);
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int64_t i = i0 + k * LPR + lr;
          if (i0 + k * LPR < e4) v[k] = i < e4 ? load(i) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);  // else not used
        }
      }
    };
    float4 v[4];
    fetch(v, 0);
    const float last = lr < (int)(cols & 3) ? x[r * cols + (e4 << 2) + lr] : 0.0f;
    if (NB == 1) {
      s.init(m, b_lo);
      s.clear();
    } else {
      constants();
    }
    for (int64_t i0 = 0; i0 < e4; i0 += 4 * LPR) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (i0 + k * LPR < e4) s.add4(v[k]);
      if (i0 + 4 * LPR < e4) fetch(v, i0 + 4 * LPR);
    }
    s.add(last);
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const float w = LPR == 16 ? row16_sum(s.total(b)) : wave_sum(s.total(b));
    if (lr == 0 && live) out[r * NB + b] = (double)w;
  }
}

// ---- per column: a lane owns 4 adjacent columns (the last lane of a row 1 to 4); the workgroup's 8
// waves take interleaved rows and meet in LDS ----
// Two workgroups per CU, so that there are few partials to fold; 12288 x 768 with the
// finishing kernel: 117 -> 27 us (16384 x 64: 128 -> 16).  half: rows a lane adds in fp32 before its sums
// go to double, at least half of its rows (the second part's way through LDS costs 12288 x 768 2.8 us of 30).
// partials: double [gridDim.y][cols][NB]
constexpr int kColWaves = 8;
template <int NB>
__global__ __launch_bounds__(kColWaves * kWave, 4) void qe_cols(const float* __restrict__ x, int64_t rows,
                                                  int64_t cols, const float* __restrict__ absmax,
                                                  int b_lo, int64_t half, double* __restrict__ partials) {
  constexpr int CPL = 4;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int64_t group = block_index();
  if (group * (kWave * CPL) >= cols) return;  // the whole workgroup
  __shared__ float lds[kColWaves * kWave * (CPL * NB + 1)];
  const int64_t c = (group * kWave + lane) * CPL;
  const int live = c + CPL <= cols ? CPL : c < cols ? (int)(cols - c) : 0;  // columns this lane owns
  // The 2 NB constants of a column cost a division each: the workgroup shares the divisions of its 256
  // columns through LDS instead of every wave forming those of its four (56 divisions per lane).
  constexpr int CST = 2 * NB + 1;  // constants of a column: 2 NB, padded to an odd pitch
  static_assert(kWave * CPL * CST <= kColWaves * kWave * (CPL * NB + 1), "the constants fit where the sums go");
  for (int i = threadIdx.x; i < kWave * CPL * NB; i += kColWaves * kWave) {
    const int cl = i / NB, b = i - cl * NB;
    const int64_t cc = group * (kWave * CPL) + cl;
    float sc = 0.0f, inv = 0.0f;
    if (cc < cols) bit_constants(absmax[cc], b_lo + b, sc, inv);
    lds[cl * CST + b] = inv;
    lds[cl * CST + NB + b] = sc;
  }
  __syncthreads();
  Sweep<NB> s[CPL];
#pragma unroll
  for (int k = 0; k < CPL; ++k) {
    s[k].m = k < live ? absmax[c + k] : 0.0f;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      s[k].inv[b] = lds[(lane * CPL + k) * CST + b];
      s[k].sc[b] = lds[(lane * CPL + k) * CST + NB + b];
      s[k].acc[b] = 0.0f;
    }
  }
  __syncthreads();  // the sums go where the constants were
  const int64_t row_step = (int64_t)gridDim.y * kColWaves;
  const int64_t r_first = (int64_t)blockIdx.y * kColWaves + wave;
  // two parts: the first one's sums wait in LDS, each lane's in its own place, until the second is done
  const bool two_parts = rows > half * row_step;
  float (*sm)[kWave][CPL * NB + 1] = reinterpret_cast<float (*)[kWave][CPL * NB + 1]>(lds);
  auto add_rows = [&](int64_t r, int64_t r_end) {
    if (live == CPL) {
#pragma unroll 2
      for (; r < r_end; r += row_step) {
        const float4 u = load_stream(x + r * cols + c);
        s[0].add(u.x); s[1].add(u.y); s[2].add(u.z); s[3].add(u.w);
      }
    } else if (live > 0) {
#pragma unroll 2
      for (; r < r_end; r += row_step) {
        const float* p = x + r * cols + c;
        const float v0 = p[0], v1 = live > 1 ? p[1] : 0.0f, v2 = live > 2 ? p[2] : 0.0f;
        s[0].add(v0); s[1].add(v1); s[2].add(v2);
      }
    }
  };
  auto put_sums = [&]() {
#pragma unroll
    for (int k = 0; k < CPL; ++k)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        sm[wave][lane][k * NB + b] = s[k].acc[b];
        s[k].acc[b] = 0.0f;
      }
  };
  if (two_parts) {
    add_rows(r_first, r_first + half * row_step < rows ? r_first + half * row_step : rows);
    put_sums();
    add_rows(r_first + half * row_step, rows);
  } else {
    add_rows(r_first, rows);
  }
  constexpr int VO = (kWave * CPL * NB + kColWaves * kWave - 1) / (kColWaves * kWave);  // sums a thread adds up
  double v[VO] = {};
  auto add_waves = [&]() {
    __syncthreads();
#pragma unroll
    for (int o = 0; o < VO; ++o) {
      const int i = threadIdx.x + o * (kColWaves * kWave);
      if (i < kWave * CPL * NB) {
        const int l = i / (CPL * NB), j = i - l * (CPL * NB);
#pragma unroll
        for (int w = 0; w < kColWaves; ++w) v[o] += (double)sm[w][l][j];
      }
    }
  };
  if (two_parts) {
    add_waves();
    __syncthreads();  // read: the second part's sums may overwrite them
  }
  put_sums();
  add_waves();
  // the workgroup's 256 columns x NB sums are consecutive in the plane of partials
  const int64_t here = (cols - group * (kWave * CPL)) * NB;
  double* dst = partials + ((int64_t)blockIdx.y * cols + group * (kWave * CPL)) * NB;
#pragma unroll
  for (int o = 0; o < VO; ++o) {
    const int i = threadIdx.x + o * (kColWaves * kWave);
    if (i < kWave * CPL * NB && i < here) dst[i] = v[o];
  }
}

// ---- per column, few rows: one launch, results written directly ------------------------------------
// A lane owns a column, the NW waves of a workgroup take interleaved rows and meet in LDS in double.  kOneRows
// rows of a wave are in flight together; their fp32 sums go to double as a whole, or two by two where one wave
// has all rows.
constexpr int kOneRows = 8;
template <int NB, int NW>
__global__ __launch_bounds__(NW * kWave) void qe_cols_one(const float* __restrict__ x, int64_t rows, int64_t cols,
                                                          const float* __restrict__ absmax, int b_lo,
                                                          double* __restrict__ out) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  __shared__ double sm[NW][kWave * NB];
  const int64_t c0 = block_index() * kWave;
  if (c0 >= cols) return;  // the whole workgroup
  const int64_t c = c0 + lane < cols ? c0 + lane : cols - 1;  // lanes past the edge: result discarded
  const float* xc = x + c;
  float v[kOneRows];
  auto fetch = [&](int64_t r) {
#pragma unroll
    for (int u = 0; u < kOneRows; ++u)
      if (r + u * NW < rows) v[u] = xc[(r + u * NW) * cols];  // wave-uniform
  };
  fetch(wave);
  Sweep<NB> s;
  if (NW == 1) {
    s.init(absmax[c], b_lo);
  } else {  // the workgroup shares the divisions of its 64 columns
    float* k = reinterpret_cast<float*>(sm[0]);
    for (int i = threadIdx.x; i < kWave * NB; i += NW * kWave) {
      const int cl = i / NB;
      float sc = 0.0f, inv = 0.0f;
      if (c0 + cl < cols) bit_constants(absmax[c0 + cl], b_lo + i - cl * NB, sc, inv);
      k[2 * i] = inv;
      k[2 * i + 1] = sc;
    }
    __syncthreads();
    s.m = absmax[c];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      s.inv[b] = k[2 * (lane * NB + b)];
      s.sc[b] = k[2 * (lane * NB + b) + 1];
      s.acc[b] = 0.0f;
    }
    __syncthreads();  // the sums go where the constants were
  }
  double a[NB] = {};
  auto flush = [&]() {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      a[b] += (double)s.acc[b];
      s.acc[b] = 0.0f;
    }
  };
  for (int64_t r = wave; r < rows; r += kOneRows * NW) {
#pragma unroll
    for (int u = 0; u < kOneRows; ++u) {
      if (r + u * NW < rows) s.add(v[u]);
      if (u == kOneRows - 1 || (NW == 1 && (u & 1))) flush();
    }
    fetch(r + kOneRows * NW);
  }
  if (NW == 1) {
    if (c0 + lane < cols) {
#pragma unroll
      for (int b = 0; b < NB; ++b) out[c * NB + b] = a[b];
    }
  } else {
#pragma unroll
    for (int b = 0; b < NB; ++b) sm[wave][lane * NB + b] = a[b];
    __syncthreads();
    const int64_t here = (cols - c0) * NB;
    for (int i = threadIdx.x; i < kWave * NB && i < here; i += NW * kWave) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) t += sm[w][i];
      out[c0 * NB + i] = t;
    }
  }
}

// ---- two-tensor squared distance -----------------------------------------------------------------
// a lane has a sum per element of a vector
struct PairSum {
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  __device__ __forceinline__ void add(float a, float b, int k = 0) { const float e = a - b; acc[k] = __builtin_fmaf(e, e, acc[k]); }
  __device__ __forceinline__ void add4(const float4& a, const float4& b) {
    add(a.x, b.x, 0); add(a.y, b.y, 1); add(a.z, b.z, 2); add(a.w, b.w, 3);
  }
};
template <bool ALIGNED, bool TILED>
__global__ __launch_bounds__(kBlock) void sse_pair_k(const float* __restrict__ y,
                                                     const float* __restrict__ yr, int64_t n,
                                                     double* __restrict__ partials) {
  PairSum s;
  const int64_t n4 = n >> 2;
  if (TILED)
    for_each_vec4_pair_tiled<ALIGNED>(reinterpret_cast<const float4*>(y), reinterpret_cast<const float4*>(yr), n4,
                             [&](const float4 a, const float4 b) { s.add4(a, b); });
  else for_each_vec4_pair_strided(y, yr, n4, [&](const float4 a, const float4 b) { s.add4(a, b); });
  const int64_t j = (n4 << 2) + threadIdx.x;  // the last n % 4 elements
  if (blockIdx.x == 0 && j < n) s.add(y[j], yr[j]);
  __shared__ double sm[kBlock / kWave];
  const double w = wave_sum_rows((s.acc[0] + s.acc[1]) + (s.acc[2] + s.acc[3]));
  if ((threadIdx.x & (kWave - 1)) == 0) sm[threadIdx.x / kWave] = w;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = (sm[0] + sm[1]) + (sm[2] + sm[3]);
}

// Up to kOnePair elements: one workgroup, one launch, lanes meet in double.  Device time, two launches against
// this: 64 x 256 4.1 / 2.4 us, 128 x 256 4.1 / 3.3.
constexpr int64_t kOnePair = 32768;
__global__ __launch_bounds__(kOneBlock) void sse_pair_one(const float* __restrict__ y, const float* __restrict__ yr,
                                                          int n, double* __restrict__ out) {
  constexpr int NW = kOneBlock / kWave;
  PairSum s;
  const int n4 = n >> 2;
#pragma unroll 4
  for (int i = threadIdx.x; i < n4; i += kOneBlock) s.add4(load4(y + 4 * i), load4(yr + 4 * i));
  if ((int)threadIdx.x < (n & 3)) s.add(y[(n & ~3) + threadIdx.x], yr[(n & ~3) + threadIdx.x]);
  __shared__ double sm[NW];
  const double w = wave_sum(((double)s.acc[0] + (double)s.acc[1]) + ((double)s.acc[2] + (double)s.acc[3]));
  if ((threadIdx.x & (kWave - 1)) == 0) sm[threadIdx.x / kWave] = w;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
#pragma unroll
    for (int v = 0; v < NW; ++v) t += sm[v];
    out[0] = t;
  }
}

// ---- launch geometry, shared by the workspace queries and the launchers --------------------------
struct QeGeom {
  unsigned gx = 1, gy = 1;
  int64_t cols_x = 1;  // per column: workgroups along the columns
  int64_t half = 1;  // per column: rows a lane adds in fp32
  int64_t nseg = 1;
  int64_t partial_doubles = 0;  // doubles of workspace
};

static QeGeom qe_geometry(int64_t rows, int64_t cols, int gran, int nb) {
  QeGeom g;
  const int64_t n = rows * cols;
  if (gran == MPQ_PER_TENSOR) {
    // 4 blocks per CU: the full sweep needs ~65 VGPRs (7 waves per SIMD), so 8 blocks per CU
    // would not be co-resident and the late blocks would trail the rest
    g.gx = flat_grid(n >> 2, kBlock * kTileVec, 4);
    const unsigned gs = flat_grid(n, kBlock * 4, 4);  // of an unaligned tensor
    g.partial_doubles = (int64_t)(g.gx > gs ? g.gx : gs) * nb;
  } else if (gran == MPQ_PER_ROW) {
    g.nseg = (cols + kSeg - 1) / kSeg;
    const int64_t blocks = (rows * g.nseg + kBlock / kWave - 1) / (kBlock / kWave);
    g.gx = (unsigned)blocks;
    g.partial_doubles = g.nseg > 1 ? rows * g.nseg * nb : 0;
  } else {
    const int64_t gx = (cols + kWave * 4 - 1) / (kWave * 4);
    // what the query has always reserved: row chunks for ~8 workgroups of 4 waves per CU, at least 8 rows
    // per wave, with 4 columns or 1 column per lane
    auto reserved = [&](int64_t gxx) {
      int64_t gy = ((int64_t)kNumCU * 8 + gxx - 1) / gxx;
      const int64_t max_gy = (rows + 4 * 8 - 1) / (4 * 8);
      if (gy > max_gy) gy = max_gy;
      if (gy < 1) gy = 1;
      if (gy > 65535) gy = 65535;
      return gy;
    };
    const int64_t r4 = reserved(gx), r1 = reserved((cols + kWave - 1) / kWave);
    g.partial_doubles = (r4 > r1 ? r4 : r1) * cols * nb;
    // what the kernel takes of it: two workgroups per CU, at least 4 rows per wave (never more than r4)
    int64_t gy = ((int64_t)kNumCU * 2 + gx - 1) / gx;
    const int64_t max_gy = (rows + kColWaves * 4 - 1) / (kColWaves * 4);
    if (gy > max_gy) gy = max_gy;
    if (gy > r4) gy = r4;
    g.cols_x = gx;
    g.gy = (unsigned)gy;
    const int64_t lane_rows = (rows + gy * kColWaves - 1) / (gy * kColWaves);
    // ... added in fp32 by a lane: no more than with one of the reserved row chunks per four waves
    const int64_t waves = 4 * ((cols & 3) == 0 ? r4 : r1), most = (rows + waves - 1) / waves;
    g.half = lane_rows <= most ? most : (lane_rows + 1) / 2;
  }
  return g;
}

// Rows that no plan holds: 16 lanes per row or a wave?  us, 16 | 64 lanes: 300 x 511 4.4 | 3.2, 1000 x 101 3.1 | 3.1,
// 1000 x 511 4.5 | 3.3, 4000 x 257 3.6 | 4.6, 4000 x 767 7.1 | 6.8, 16384 x 1023 16.2 | 20.2, 16384 x 2047 26.8 | 28.1; one
// width 4000 x 257 2.6 | 2.9, 4000 x 511 3.9 | 3.7, 16384 x 511 6.4 | 8.0, 16384 x 1023 12.9 | 12.1.
static bool qe_rows_short(int64_t rows, int64_t cols, int nb) {
  if (rows >= 8192) return cols <= (nb < 3 ? 768 : 2048);
  return cols <= 64 || cols <= rows / 8;
}

// Waves of a workgroup of qe_cols_one, 0 where qe_cols and its finishing kernel are faster (groups: of 64 columns).
// us for seven widths, 1 | 4 | 16 waves / two launches: 8 x 4096 3.2 | 3.5 | 3.6 / 7.1, 32 x 4096 5.7 | 3.8 | 4.0 / 8.5,
// 64 x 300001 25.9 | 30.3 | 61 / 60, 64 x 65536 11.6 | 8.0 | 14.5 / 18, 256 x 101 28.8 | 9.5 | 5.9 / 7.3, 512 x 16384
// 59 | 20 | 10.4 / 20, 512 x 64 - | 16 | 8.8 / 9, 1000 x 64 - | 30 | 14.5 / 8, 1000 x 4096 - | 31 | 15.3 / 16.
static int qe_cols_waves(int64_t rows, int64_t groups) {
  if (rows <= 8 || (rows <= 64 && groups >= 2048)) return 1;
  if (rows <= 32 || (rows <= 512 && groups >= 512)) return 4;
  return rows <= 512 ? 16 : 0;
}

template <int NB>
static void launch_qe(const QeGeom& g, const float* x, int64_t rows, int64_t cols, int gran,
                      const float* absmax, int b_lo, double* out, double* ws, hipStream_t st) {
  const int64_t n = rows * cols;
  if (gran == MPQ_PER_TENSOR && n * NB <= kOneLimit && n <= (aligned16(x) ? kOneMost : kOneMost / 4)) {
    qe_one<NB><<<1, kOneBlock, 0, st>>>(x, (int)n, absmax, b_lo, out);
  } else if (gran == MPQ_PER_TENSOR) {
    unsigned parts = g.gx;
    if (aligned16(x)) {
      qe_flat<NB, true, true><<<parts, kBlock, 0, st>>>(x, n, absmax, b_lo, ws);
    } else if (n > kTiledFrom) {
      qe_flat<NB, false, true><<<parts, kBlock, 0, st>>>(x, n, absmax, b_lo, ws);
    } else {
      parts = flat_grid(n, kBlock * 4, 4);
      qe_flat<NB, false, false><<<parts, kBlock, 0, st>>>(x, n, absmax, b_lo, ws);
    }
    qe_finish_tree<NB><<<1, kBlock, 0, st>>>(ws, (int64_t)parts, out);
  } else if (gran == MPQ_PER_ROW) {
    if (g.nseg == 1) {
      const bool plan_holds = (cols & 3) == 0 && aligned16(x);
      // (the batched kernels': 16 lanes per row up to 2048 columns, else a wave)
      const bool sixteen = plan_holds ? cols <= 2048 : qe_rows_short(rows, cols, NB);
      const int64_t per = sixteen ? kBlock / 16 : kBlock / kWave;
      const unsigned blocks = (unsigned)((rows + per - 1) / per);
      if (plan_holds && sixteen) qe_rows_sub<NB, 16, true><<<blocks, kBlock, 0, st>>>(x, rows, cols, absmax, b_lo, out);
      else if (plan_holds) qe_rows_sub<NB, 64, true><<<blocks, kBlock, 0, st>>>(x, rows, cols, absmax, b_lo, out);
      else if (sixteen) qe_rows_sub<NB, 16, false><<<blocks, kBlock, 0, st>>>(x, rows, cols, absmax, b_lo, out);
      else qe_rows_sub<NB, 64, false><<<blocks, kBlock, 0, st>>>(x, rows, cols, absmax, b_lo, out);
    } else {
      qe_rows<NB><<<g.gx, kBlock, 0, st>>>(x, rows, cols, g.nseg, absmax, b_lo, ws);
      const int64_t k = rows * NB;
      qe_finish_planes<<<wide_grid((k + kWave - 1) / kWave, kBlock), kBlock, 0, st>>>(ws, rows, g.nseg, NB, g.nseg * NB, NB, out);
    }
  } else {
    const int64_t groups = (cols + kWave - 1) / kWave;
    const int nw = qe_cols_waves(rows, groups);
    if (nw == 16) {
      qe_cols_one<NB, 16><<<wide_grid(groups, 16 * kWave), 16 * kWave, 0, st>>>(x, rows, cols, absmax, b_lo, out);
      return;
    }
    if (nw == 4) {
      qe_cols_one<NB, 4><<<wide_grid(groups, 4 * kWave), 4 * kWave, 0, st>>>(x, rows, cols, absmax, b_lo, out);
      return;
    }
    if (nw == 1) {
      qe_cols_one<NB, 1><<<wide_grid(groups, kWave), kWave, 0, st>>>(x, rows, cols, absmax, b_lo, out);
      return;
    }
    qe_cols<NB><<<wide_grid(g.cols_x, kColWaves * kWave, g.gy), kColWaves * kWave, 0, st>>>(x, rows, cols, absmax, b_lo, g.half, ws);
    const int64_t k = cols * NB;
    qe_finish_planes<<<wide_grid((k + kWave - 1) / kWave, kBlock), kBlock, 0, st>>>(ws, cols, (int64_t)g.gy, NB, NB, cols * NB, out);
  }
}

static int check_qe_args(int64_t rows, int64_t cols, int gran, int b_lo, int b_hi) {
  if (rows <= 0 || cols <= 0 || mul_overflows(rows, cols)) return MPQ_ERR_SHAPE;
  if (gran < MPQ_PER_TENSOR || gran > MPQ_PER_COL) return MPQ_ERR_GRAN;
  if (b_lo < 2 || b_hi > 8 || b_lo > b_hi) return MPQ_ERR_BITS;
  if (gran == MPQ_PER_ROW && (rows * ((cols + kSeg - 1) / kSeg) + 3) / 4 > 0x7FFFFFFF) return MPQ_ERR_SHAPE;
  if (gran == MPQ_PER_COL && (cols + kWave - 1) / kWave > 0x7FFFFFFF) return MPQ_ERR_SHAPE;
  return MPQ_OK;
}

}  // namespace mpq

using namespace mpq;

extern "C" size_t mpq_quant_error_workspace_bytes(int64_t rows, int64_t cols, int gran, int b_lo,
                                                  int b_hi) {
  if (check_qe_args(rows, cols, gran, b_lo, b_hi) != MPQ_OK) return 0;
  const QeGeom g = qe_geometry(rows, cols, gran, b_hi - b_lo + 1);
  return (size_t)g.partial_doubles * sizeof(double);
}

static int run_quant_error(const float* x, int64_t rows, int64_t cols, int gran, const float* absmax, int b_lo,
                           int b_hi, double* sse_out, void* ws, size_t ws_bytes, bool builtin_scratch,
                           void* stream) {
  if (!x || !absmax || !sse_out) return MPQ_ERR_NULL;
  const int rc = check_qe_args(rows, cols, gran, b_lo, b_hi);
  if (rc != MPQ_OK) return rc;
  const int nb = b_hi - b_lo + 1;
  const QeGeom g = qe_geometry(rows, cols, gran, nb);
  const size_t need = (size_t)g.partial_doubles * sizeof(double);
  if (need > 0 && (!ws || ws_bytes < need)) return builtin_scratch ? MPQ_ERR_TOO_LARGE : MPQ_ERR_WORKSPACE;
  if (need > 0 && !aligned16(ws)) return MPQ_ERR_ALIGN;
  if ((reinterpret_cast<uintptr_t>(sse_out) & 7u) != 0) return MPQ_ERR_ALIGN;
  hipStream_t st = (hipStream_t)stream;
  double* wsd = reinterpret_cast<double*>(ws);
  switch (nb) {
    case 1: launch_qe<1>(g, x, rows, cols, gran, absmax, b_lo, sse_out, wsd, st); break;
    case 2: launch_qe<2>(g, x, rows, cols, gran, absmax, b_lo, sse_out, wsd, st); break;
    case 3: launch_qe<3>(g, x, rows, cols, gran, absmax, b_lo, sse_out, wsd, st); break;
    case 4: launch_qe<4>(g, x, rows, cols, gran, absmax, b_lo, sse_out, wsd, st); break;
    case 5: launch_qe<5>(g, x, rows, cols, gran, absmax, b_lo, sse_out, wsd, st); break;
    case 6: launch_qe<6>(g, x, rows, cols, gran, absmax, b_lo, sse_out, wsd, st); break;
    default: launch_qe<7>(g, x, rows, cols, gran, absmax, b_lo, sse_out, wsd, st); break;
  }
  return launch_status();
}

extern "C" int mpq_quant_error(const float* x, int64_t rows, int64_t cols, int gran,
                               const float* absmax, int b_lo, int b_hi, double* sse_out, void* ws,
                               size_t ws_bytes, void* stream) {
  return run_quant_error(x, rows, cols, gran, absmax, b_lo, b_hi, sse_out, ws, ws_bytes, false, stream);
}

// ---- the sweep for callers that cannot allocate -------------------------------------------------
// The partial sums live in a buffer that is part of the library's device image, so the call needs
// neither a workspace from the caller nor any allocation.  Every GPU the library runs on holds its
// own copy of the buffer, at its own address, for the life of the process.  In host code the
// array's name is only a handle for hipGetSymbolAddress: the device address is looked up once per
// device (with that device current) and kept; everything that touches the memory uses that pointer.
constexpr size_t kScratchBytes = MPQ_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// device address of `scratch` on the current device
int scratch_of_current_device(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    set_last_hip_error((int)(e != hipSuccess ? e : hipErrorInvalidDevice));
    return MPQ_ERR_HIP;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      set_last_hip_error((int)(e != hipSuccess ? e : hipErrorInvalidSymbol));
      return MPQ_ERR_HIP;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return MPQ_OK;
}
}  // namespace

extern "C" int mpq_quant_error_noalloc(const float* x, int64_t rows, int64_t cols, int gran, const float* absmax,
                                       int b_lo, int b_hi, double* sse_out, void* stream) {
  // arguments first: a call that cannot succeed must not touch the device at all
  if (!x || !absmax || !sse_out) return MPQ_ERR_NULL;
  int rc = check_qe_args(rows, cols, gran, b_lo, b_hi);
  if (rc != MPQ_OK) return rc;
  if (mpq_quant_error_workspace_bytes(rows, cols, gran, b_lo, b_hi) > kScratchBytes) return MPQ_ERR_TOO_LARGE;
  void* ptr = nullptr;
  rc = scratch_of_current_device(&ptr);
  if (rc != MPQ_OK) return rc;
  // every partial the finishing kernel reads is written by the main kernel of the same call:
  // nothing in the buffer has to start at zero
  return run_quant_error(x, rows, cols, gran, absmax, b_lo, b_hi, sse_out, ptr, kScratchBytes, true, stream);
}

extern "C" size_t mpq_sse_pair_workspace_bytes(int64_t n) {
  if (n <= 0 || n > ((int64_t)1 << 46)) return 0;
  const unsigned a = flat_grid(n >> 2, kBlock * 2), b = flat_grid(n, kBlock * 4);
  return (size_t)(a > b ? a : b) * sizeof(double);
}

extern "C" int mpq_sse_pair(const float* y, const float* y_ref, int64_t n, double* sse_out,
                            void* ws, size_t ws_bytes, void* stream) {
  if (!y || !y_ref || !sse_out) return MPQ_ERR_NULL;
  if (n <= 0 || n > ((int64_t)1 << 46)) return MPQ_ERR_SHAPE;
  if (!ws || ws_bytes < mpq_sse_pair_workspace_bytes(n)) return MPQ_ERR_WORKSPACE;
  if (!aligned16(ws) || (reinterpret_cast<uintptr_t>(sse_out) & 7u) != 0) return MPQ_ERR_ALIGN;
  hipStream_t st = (hipStream_t)stream;
  if (n <= kOnePair) {
    sse_pair_one<<<1, kOneBlock, 0, st>>>(y, y_ref, (int)n, sse_out);
    return launch_status();
  }
  double* wsd = reinterpret_cast<double*>(ws);
  const bool aligned = aligned16(y) && aligned16(y_ref);
  const bool tiled = aligned || n > kTiledFrom;
  const unsigned grid = tiled ? flat_grid(n >> 2, kBlock * 2) : flat_grid(n, kBlock * 4);
  if (aligned) sse_pair_k<true, true><<<grid, kBlock, 0, st>>>(y, y_ref, n, wsd);
  else if (tiled) sse_pair_k<false, true><<<grid, kBlock, 0, st>>>(y, y_ref, n, wsd);
  else sse_pair_k<false, false><<<grid, kBlock, 0, st>>>(y, y_ref, n, wsd);
  qe_finish_tree<1><<<1, kBlock, 0, st>>>(wsd, (int64_t)grid, sse_out);
  return launch_status();
}
