// scale_adjust.hip -- the adjustment step of Sec. 3.1: after max calibration the two scales of
// Eq. 1 are free parameters and are moved by gradient descent while the model's own parameters
// stay put.  In the integer form used throughout this library the pair is
//   inv   (= alpha * levels): applied before rounding,     code = clamp(RNE(x * inv), +-qmax)
//   scale (= gamma / levels): applied after,                Q = code * scale
// and calibration sets inv = qmax / m, scale = m / qmax.
//
// Gradients treat rounding as the identity (straight-through): with g = dL/dQ
//   dL/dscale = sum g * code
//   dL/dinv   = scale * sum over elements whose rounded value needs no clamping of g * x
// g == NULL selects the reconstruction loss L = sum (Q - x)^2, g = 2 (Q - x).
//
// code for arbitrary inv: x is first clamped to +-2^20 / |inv| so that the magic-number rounding
// (exact product rounded to nearest even by one fused add of 1.5 * 2^23) stays in its valid range;
// 2^20 is far beyond qmax + 1/2, so neither the code nor the "needs no clamping" test changes.
#include "common.hpp"

#include <type_traits>

namespace mpq {

struct TwoScales {
  float inv, scale, lim, qmax;
  __device__ __forceinline__ TwoScales(float inv_, float scale_, int bits) : inv(inv_), scale(scale_) {
    qmax = (float)((1 << (bits - 1)) - 1);
    lim = 1048576.0f / fabsf(inv_);  // +inf for inv == 0: nothing to clamp, every product is 0
  }
  // rounded value before clamping, as an integer-valued float
  __device__ __forceinline__ float rounded(float x) const {
    const float xc = __builtin_amdgcn_fmed3f(x, -lim, lim);
    return __builtin_fmaf(xc, inv, kMagic) - kMagic;
  }
};

// lane-local sums of one element's contributions
struct GradAcc {
  float s_code = 0.0f, s_x = 0.0f, s_loss = 0.0f;
  template <bool HAS_G>
  __device__ __forceinline__ void add(const TwoScales& t, float x, float g_in) {
    const float r = t.rounded(x);
    const float q = __builtin_amdgcn_fmed3f(r, -t.qmax, t.qmax);
    const float e = __builtin_fmaf(q, t.scale, -x);
    const float g = HAS_G ? g_in : 2.0f * e;
    s_code = __builtin_fmaf(g, q, s_code);
    if (r == q) s_x = __builtin_fmaf(g, x, s_x);  // the clamp was inactive
    s_loss = __builtin_fmaf(e, e, s_loss);
  }
};

// One for each of the four elements of a vector, which keeps the fp32 chains short.
template <bool HAS_G>
struct GradAcc4 {
  GradAcc k[4];
  __device__ __forceinline__ void add(const TwoScales& t, float x, float g) { k[0].template add<HAS_G>(t, x, g); }
  __device__ __forceinline__ void add4(const TwoScales& t, const float4& v, const float4& g) {
    k[0].template add<HAS_G>(t, v.x, g.x);
    k[1].template add<HAS_G>(t, v.y, g.y);
    k[2].template add<HAS_G>(t, v.z, g.z);
    k[3].template add<HAS_G>(t, v.w, g.w);
  }
  __device__ __forceinline__ float code() const { return (k[0].s_code + k[1].s_code) + (k[2].s_code + k[3].s_code); }
  __device__ __forceinline__ float x() const { return (k[0].s_x + k[1].s_x) + (k[2].s_x + k[3].s_x); }
  __device__ __forceinline__ float loss() const { return (k[0].s_loss + k[1].s_loss) + (k[2].s_loss + k[3].s_loss); }
};

// One for all of them: where a lane has one vector, the products' own roundings count (a sum's first product is
// rounded, the others enter it exactly: dscale of 1000 x 64 per row 1.31e-8 of the sum of absolute values against
// 1.36e-8, of 3200 x 112 per tensor 3.4e-9 against 8.1e-9).
template <bool HAS_G>
struct GradAcc1 {
  GradAcc k;
  __device__ __forceinline__ void add(const TwoScales& t, float x, float g) { k.template add<HAS_G>(t, x, g); }
  __device__ __forceinline__ void add4(const TwoScales& t, const float4& v, const float4& g) {
    add(t, v.x, g.x); add(t, v.y, g.y); add(t, v.z, g.z); add(t, v.w, g.w);
  }
  __device__ __forceinline__ float code() const { return k.s_code; }
  __device__ __forceinline__ float x() const { return k.s_x; }
  __device__ __forceinline__ float loss() const { return k.s_loss; }
};

// ---- per tensor: one partial triple per workgroup ----------------------------------------------
// TILED: tiles dealt round-robin, else (small tensors) one vector a trip
template <bool HAS_G, bool TILED, bool STREAM>
__global__ __launch_bounds__(kBlock) void sg_flat(const float* __restrict__ x, const float* __restrict__ g,
                                                  int64_t n, const float* __restrict__ inv,
                                                  const float* __restrict__ scale, int bits,
                                                  double* __restrict__ partials) {
  const TwoScales t(inv[0], scale[0], bits);
  std::conditional_t<TILED, GradAcc4<HAS_G>, GradAcc1<HAS_G>> a;
  const int64_t n4 = n >> 2;
  if (TILED) {
    if (HAS_G)
      for_each_vec4_pair_tiled<STREAM>(reinterpret_cast<const float4*>(x), reinterpret_cast<const float4*>(g), n4,
                               [&](const float4 v, const float4 u) { a.add4(t, v, u); });
    else
      for_each_vec4_tiled<STREAM>(reinterpret_cast<const float4*>(x), n4, [&](const float4 v, int64_t) { a.add4(t, v, v); });
  } else {
    if (HAS_G) for_each_vec4_pair_strided(x, g, n4, [&](const float4 v, const float4 u) { a.add4(t, v, u); });
    else for_each_vec4_strided(x, n4, [&](const float4 v) { a.add4(t, v, v); });
  }
  const int64_t j = (n4 << 2) + threadIdx.x;  // the last n % 4 elements
  if (blockIdx.x == 0 && j < n) a.add(t, x[j], HAS_G ? g[j] : 0.0f);
  __shared__ double sm[3][kBlock / kWave];
  const double w0 = wave_sum_rows(a.code()), w1 = wave_sum_rows(a.x()), w2 = wave_sum_rows(a.loss());
  if ((threadIdx.x & (kWave - 1)) == 0) {
    sm[0][threadIdx.x / kWave] = w0;
    sm[1][threadIdx.x / kWave] = w1;
    sm[2][threadIdx.x / kWave] = w2;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const double* s = sm[threadIdx.x];
    partials[(int64_t)blockIdx.x * 3 + threadIdx.x] = (s[0] + s[1]) + (s[2] + s[3]);
  }
}

// one workgroup folds the partial triples in a fixed order and applies the factor of dL/dinv
__global__ __launch_bounds__(kBlock) void sg_finish(const double* __restrict__ partials, int64_t count,
                                                    const float* __restrict__ scale, double* __restrict__ dinv,
                                                    double* __restrict__ dscale, double* __restrict__ loss) {
  __shared__ double sm[3][kBlock];
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  for (int64_t i = threadIdx.x; i < count; i += kBlock) {
    a0 += partials[i * 3];
    a1 += partials[i * 3 + 1];
    a2 += partials[i * 3 + 2];
  }
  sm[0][threadIdx.x] = a0;
  sm[1][threadIdx.x] = a1;
  sm[2][threadIdx.x] = a2;
  __syncthreads();
  for (int h = kBlock / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h)
      for (int k = 0; k < 3; ++k) sm[k][threadIdx.x] += sm[k][threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    dscale[0] = sm[0][0];
    dinv[0] = (double)scale[0] * sm[1][0];
    if (loss) loss[0] = sm[2][0];
  }
}

// ---- per row: LPR lanes per row (16 or 64), results written directly ------------------------------
// U 16-byte loads per tensor in flight per lane, the first ones in front of the scales: four where a row has
// several trips for them (12288 x 768 9.8 -> 8.9 us, with a gradient 13.7 -> 12.5), one where the code's length
// counts, as it is fetched cold (300 x 256 2.9 -> 2.4).
template <typename Acc, bool HAS_G, int LPR, int U, bool STREAM>
__global__ __launch_bounds__(kBlock) void sg_rows(const float* __restrict__ x, const float* __restrict__ g,
                                                  int64_t rows, int64_t cols, const float* __restrict__ inv,
                                                  const float* __restrict__ scale, int bits,
                                                  double* __restrict__ dinv, double* __restrict__ dscale,
                                                  double* __restrict__ loss) {
  const int lr = threadIdx.x % LPR;
  int64_t r = (int64_t)blockIdx.x * (kBlock / LPR) + threadIdx.x / LPR;
  const bool live = r < rows;
  if (!live) r = rows - 1;  // every lane stays active for the cross-lane sums; result discarded
  const float* xr = x + r * cols;
  const float* gr = HAS_G ? g + r * cols : nullptr;
  constexpr int64_t kStep = 4 * LPR;
  float4 v[U], u[U];
  auto fetch = [&](int64_t c0) {
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int64_t c = c0 + k * kStep + 4 * lr;
      if (c + 4 <= cols) {
        v[k] = STREAM ? load_stream(xr + c) : load4(xr + c);
        if (HAS_G) u[k] = STREAM ? load_stream(gr + c) : load4(gr + c);
      }
    }
  };
  fetch(0);
  const bool tail = lr < (int)(cols & 3);
  const int64_t e = (cols & ~(int64_t)3) + lr;
  const float xe = tail ? xr[e] : 0.0f, ge = HAS_G && tail ? gr[e] : 0.0f;
  const TwoScales t(inv[r], scale[r], bits);
  Acc a;
#pragma unroll 1
  for (int64_t c0 = 0; c0 + 4 <= cols; c0 += U * kStep) {  // the same trips for every lane of the row
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (c0 + k * kStep + 4 * lr + 4 <= cols) a.add4(t, v[k], HAS_G ? u[k] : v[k]);
    fetch(c0 + U * kStep);
  }
  if (tail) a.add(t, xe, ge);
  const float w0 = LPR == 16 ? row16_sum(a.code()) : wave_sum(a.code());
  const float w1 = LPR == 16 ? row16_sum(a.x()) : wave_sum(a.x());
  const float w2 = LPR == 16 ? row16_sum(a.loss()) : wave_sum(a.loss());
  if (lr == 0 && live) {
    dscale[r] = (double)w0;
    dinv[r] = (double)t.scale * (double)w1;
    if (loss) loss[r] = (double)w2;
  }
}

// ---- forward with explicit scales ----------------------------------------------------------------
// One thread per element with a division per element for its row and another for the clamp's limit
// took 28 us on 12288 x 768 and 185 on 16384 x 4096; sixteen bytes at a time, the limit once per lane and row,
// 14.5 and 81.
__device__ __forceinline__ float q_of(const TwoScales& t, float x) {
  return __builtin_amdgcn_fmed3f(t.rounded(x), -t.qmax, t.qmax);
}
typedef unsigned u32_any __attribute__((aligned(1)));  // codes may start at any byte

// four outputs from flat element e on
__device__ __forceinline__ void fqs_emit4(const TwoScales& t, const float4& v, int64_t e, float* y, int8_t* codes) {
  const float q0 = q_of(t, v.x), q1 = q_of(t, v.y), q2 = q_of(t, v.z), q3 = q_of(t, v.w);
  if (y) store4(y + e, make_float4(q0 * t.scale, q1 * t.scale, q2 * t.scale, q3 * t.scale));
  if (codes)
    *reinterpret_cast<u32_any*>(codes + e) = ((unsigned)(int)q0 & 0xFFu) | (((unsigned)(int)q1 & 0xFFu) << 8) |
                                             (((unsigned)(int)q2 & 0xFFu) << 16) | ((unsigned)(int)q3 << 24);
}
__device__ __forceinline__ void fqs_emit1(const TwoScales& t, float v, int64_t e, float* y, int8_t* codes) {
  const float q = q_of(t, v);
  if (y) y[e] = q * t.scale;
  if (codes) codes[e] = (int8_t)(int)q;
}

__global__ __launch_bounds__(kBlock) void fqs_flat(const float* __restrict__ x, int64_t n, const float* __restrict__ inv,
                                                   const float* __restrict__ scale, int bits, float* __restrict__ y,
                                                   int8_t* __restrict__ codes) {
  const TwoScales t(inv[0], scale[0], bits);
  const int64_t n4 = n >> 2;
  for_each_vec4_tiled(reinterpret_cast<const float4*>(x), n4,
                      [&](const float4 v, int64_t i) { fqs_emit4(t, v, i << 2, y, codes); });
  const int64_t j = (n4 << 2) + threadIdx.x;  // the last n % 4 elements
  if (blockIdx.x == 0 && j < n) fqs_emit1(t, x[j], j, y, codes);
}

// LPR lanes per row (4, 16 or 64); blockIdx.y: segments of seg columns (a multiple of 4)
template <int LPR>
__global__ __launch_bounds__(kBlock) void fqs_rows(const float* __restrict__ x, int64_t rows, int64_t cols,
                                                   const float* __restrict__ inv, const float* __restrict__ scale,
                                                   int bits, int64_t seg, float* __restrict__ y,
                                                   int8_t* __restrict__ codes) {
  const int lr = threadIdx.x % LPR;
  const int64_t r = block_index() * (kBlock / LPR) + threadIdx.x / LPR;
  if (r >= rows) return;
  const TwoScales t(inv[r], scale[r], bits);
  const int64_t c0 = (int64_t)blockIdx.y * seg, c1 = c0 + seg < cols ? c0 + seg : cols;
  const int64_t end = r * cols + c1;
  constexpr int64_t kStep = 4 * LPR;
  for (int64_t i = r * cols + c0 + 4 * lr; i + 4 <= end; i += 4 * kStep) {  // four loads in flight per lane
    float4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i + k * kStep + 4 <= end) v[k] = LPR == kWave ? load_stream(x + i + k * kStep) : load4(x + i + k * kStep);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i + k * kStep + 4 <= end) fqs_emit4(t, v[k], i + k * kStep, y, codes);
  }
  const int64_t e = end - (c1 & 3) + lr;
  if (e < end) fqs_emit1(t, x[e], e, y, codes);
}

// ---- p <- fl32(p - lr * dL/dp), in double, rounded once -----------------------------------------
__global__ void sgd_k(float* __restrict__ inv, float* __restrict__ scale, const double* __restrict__ dinv,
                      const double* __restrict__ dscale, int64_t count, double lr) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  inv[i] = (float)((double)inv[i] - lr * dinv[i]);
  scale[i] = (float)((double)scale[i] - lr * dscale[i]);
}

static int check_sa(int64_t rows, int64_t cols, int gran, int bits) {
  if (rows <= 0 || cols <= 0 || mul_overflows(rows, cols)) return MPQ_ERR_SHAPE;
  if (gran != MPQ_PER_TENSOR && gran != MPQ_PER_ROW) return MPQ_ERR_GRAN;
  if (bits < 2 || bits > 8) return MPQ_ERR_BITS;
  if (gran == MPQ_PER_ROW && (rows + 3) / 4 > 0x7FFFFFFF) return MPQ_ERR_SHAPE;
  return MPQ_OK;
}

static unsigned sg_grid(int64_t n, bool has_g) { return flat_grid(n >> 2, kBlock * (has_g ? 2 : kTileVec)); }

// Gradients per row: 16 lanes per row or a wave?  us with an upstream gradient, 16 | 64 lanes: 1000 x 101 2.6 | 2.5,
// 5000 x 101 2.9 | 3.2, 5000 x 255 4.3 | 4.1, 16384 x 384 9.9 | 10.5, 16384 x 511 13.7 | 12.3, 40000 x 384 20.2 | 20.6.
static bool sg_sixteen(int64_t rows, int64_t cols) { return cols <= 64 || cols <= rows / 32; }
// Tensors beyond the caches are streamed: 16384 x 768 with a gradient 18.5 -> 16.9 us, but 1000 x 4096 9.3 -> 11.8.
constexpr int64_t kStreamFrom = 5ll << 20;

// Forward: rows of up to kShortRow columns are walked by 16 lanes each, longer ones by a wave: 16 against 64
// lanes, 3001 x 1147 9.8 / 7.5 us.
constexpr int64_t kShortRow = 256;

}  // namespace mpq

using namespace mpq;

extern "C" int mpq_fake_quant_scales(const float* x, int64_t rows, int64_t cols, int gran, const float* inv,
                                     const float* scale, int bits, float* y_out, int8_t* codes_out,
                                     void* stream) {
  if (!x || !inv || !scale || (!y_out && !codes_out)) return MPQ_ERR_NULL;
  const int rc = check_sa(rows, cols, gran, bits);
  if (rc != MPQ_OK) return rc;
  hipStream_t st = (hipStream_t)stream;
  if (gran == MPQ_PER_TENSOR)
    fqs_flat<<<flat_grid((rows * cols) >> 2, kBlock * kTileVec), kBlock, 0, st>>>(x, rows * cols, inv, scale, bits, y_out, codes_out);
  else if (cols <= 32)
    fqs_rows<4><<<wide_grid((rows + 63) / 64, kBlock), kBlock, 0, st>>>(x, rows, cols, inv, scale, bits, cols, y_out, codes_out);
  else if (cols <= kShortRow)
    fqs_rows<16><<<wide_grid((rows + 15) / 16, kBlock), kBlock, 0, st>>>(x, rows, cols, inv, scale, bits, cols, y_out, codes_out);
  else {
    // few long rows: cut into segments of whole trips (1024 columns a wave) until the chip has its waves
    int64_t nseg = (2048 + rows - 1) / rows;
    if (nseg > (cols + 1023) / 1024) nseg = (cols + 1023) / 1024;
    const int64_t seg = ((cols + nseg - 1) / nseg + 1023) / 1024 * 1024;
    const dim3 grid = wide_grid((rows + 3) / 4, kBlock, (unsigned)((cols + seg - 1) / seg));
    fqs_rows<64><<<grid, kBlock, 0, st>>>(x, rows, cols, inv, scale, bits, seg, y_out, codes_out);
  }
  return launch_status();
}

extern "C" size_t mpq_scale_grad_workspace_bytes(int64_t rows, int64_t cols, int gran) {
  if (check_sa(rows, cols, gran, 8) != MPQ_OK || gran != MPQ_PER_TENSOR) return 0;
  const int64_t n = rows * cols;
  unsigned g = flat_grid(n, kBlock * 4);  // the grid of small tensors
  for (int v = 0; v < 2; ++v) {           // ... and for the largest grid any variant may use
    const unsigned c = sg_grid(n, v != 0);
    g = c > g ? c : g;
  }
  return (size_t)g * 3 * sizeof(double);
}

extern "C" int mpq_scale_grad(const float* x, int64_t rows, int64_t cols, int gran, const float* inv,
                              const float* scale, int bits, const float* g, double* dinv_out,
                              double* dscale_out, double* loss_out, void* ws, size_t ws_bytes, void* stream) {
  if (!x || !inv || !scale || !dinv_out || !dscale_out) return MPQ_ERR_NULL;
  const int rc = check_sa(rows, cols, gran, bits);
  if (rc != MPQ_OK) return rc;
  if ((reinterpret_cast<uintptr_t>(dinv_out) | reinterpret_cast<uintptr_t>(dscale_out) |
       reinterpret_cast<uintptr_t>(loss_out)) & 7u)
    return MPQ_ERR_ALIGN;
  hipStream_t st = (hipStream_t)stream;
  const int64_t n = rows * cols;
  if (gran == MPQ_PER_TENSOR) {
    if (!ws || ws_bytes < mpq_scale_grad_workspace_bytes(rows, cols, gran)) return MPQ_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(ws) & 7u) return MPQ_ERR_ALIGN;
    double* partials = reinterpret_cast<double*>(ws);
    // below kTiledFrom tiles give too few CUs a workgroup: 255000 4.7 us against 5.4, but 1000001 6.2 against 5.8
    const bool tiled = n > kTiledFrom, aligned = aligned16(x) && (!g || aligned16(g));
    const unsigned grid = tiled ? sg_grid(n, g != nullptr) : flat_grid(n, kBlock * 4);
#define MPQ_SG(G_) \
  (!tiled ? sg_flat<G_, false, false><<<grid, kBlock, 0, st>>>(x, g, n, inv, scale, bits, partials) \
   : aligned ? sg_flat<G_, true, true><<<grid, kBlock, 0, st>>>(x, g, n, inv, scale, bits, partials) \
             : sg_flat<G_, true, false><<<grid, kBlock, 0, st>>>(x, g, n, inv, scale, bits, partials))
    if (g) MPQ_SG(true);
    else MPQ_SG(false);
#undef MPQ_SG
    sg_finish<<<1, kBlock, 0, st>>>(partials, (int64_t)grid, scale, dinv_out, dscale_out, loss_out);
  } else {
    const bool sixteen = sg_sixteen(rows, cols), short_code = cols <= (sixteen ? 256 : 768), stream = rows * cols > kStreamFrom;
    const unsigned grid = (unsigned)(sixteen ? (rows + 15) / 16 : (rows + 3) / 4);
#define MPQ_SG(ACC_, G_, LPR_, U_, S_) \
  sg_rows<ACC_<G_>, G_, LPR_, U_, S_><<<grid, kBlock, 0, st>>>(x, g, rows, cols, inv, scale, bits, dinv_out, dscale_out, loss_out)
#define MPQ_SG_U(G_, LPR_)                                             \
  if (stream) MPQ_SG(GradAcc4, G_, LPR_, 4, true);                     \
  else if (cols < 4 * LPR_ + 4) MPQ_SG(GradAcc1, G_, LPR_, 1, false);  \
  else if (short_code) MPQ_SG(GradAcc4, G_, LPR_, 1, false);           \
  else MPQ_SG(GradAcc4, G_, LPR_, 4, false)
    if (sixteen) {
      if (g) { MPQ_SG_U(true, 16); }
      else { MPQ_SG_U(false, 16); }
    } else {
      if (g) { MPQ_SG_U(true, 64); }
      else { MPQ_SG_U(false, 64); }
    }
#undef MPQ_SG_U
#undef MPQ_SG
  }
  return launch_status();
}

extern "C" int mpq_scale_sgd_step(float* inv, float* scale, const double* dinv, const double* dscale,
                                  int64_t count, double lr, void* stream) {
  if (!inv || !scale || !dinv || !dscale) return MPQ_ERR_NULL;
  if (count <= 0 || (count + 255) / 256 > 0x7FFFFFFF) return MPQ_ERR_SHAPE;
  sgd_k<<<(unsigned)((count + 255) / 256), 256, 0, (hipStream_t)stream>>>(inv, scale, dinv, dscale, count, lr);
  return launch_status();
}
