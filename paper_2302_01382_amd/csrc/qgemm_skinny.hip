// qgemm_skinny.hip -- the quantized linear layer where the output has few tiles (any layer at inference
// batch 1, small layers): one launch, no LDS tiles, k split over the waves of a workgroup.
//
// What bounds such a layer is latency: a 49 x 4608 x 512 layer is 2.4 MB of operands, well under a
// microsecond of memory time, but a 64 x 64 tile walks its 36 k tiles one barrier after the other on 8
// of the 256 CUs.  Here the output is cut into 16 x 16 tiles, so that more CUs have one, and the waves
// of a workgroup deal the k steps of 128 out between them.  Both operands are K-contiguous, which is
// the operand layout of v_mfma_i32_16x16x64_i8, so a lane loads its operands straight into registers
// (the order of k inside a dot product is free as long as both operands agree).  A wave's loads of
// four steps are in flight before its first matrix step.  The waves' accumulators meet in LDS
// (integers: exact in any order).  Loads go to any byte address (load_chunk16), so K and the pointers
// need no alignment.  Packed int4 next to int8 in brackets, us (M x K x N): 49 x 4608 x 512 split along k
// in two launches 8.7 -> 6.7 (8.9 -> 5.7), 49 x 1024 x 512 6.3 -> 3.7 (6.6 -> 3.4), 64 x 256 x 256 in
// 64 x 64 tiles 3.9 -> 3.0 (4.0 -> 2.9).  A 32 x 32 tile per workgroup (half the operand bytes per output)
// is slower wherever this kernel is taken (49 x 4608 x 512: 11) as fewer CUs have one; sixteen waves spill.
#include "qgemm_dma.hpp"

namespace mpq {

// NW: waves, which split k
template <int NW, bool W4>
__global__ __launch_bounds__(NW * 64) void qgemm_skinny(const int8_t* __restrict__ A, const void* __restrict__ Wv,
                                                        int64_t M, int64_t N, int64_t K,
                                                        const float* __restrict__ a_scale,
                                                        const float* __restrict__ w_scale, int w_per_row,
                                                        float* __restrict__ Y, int32_t* __restrict__ ACC,
                                                        EpiArgs epi, int vec) {
  constexpr int U = 4;            // k steps whose loads are in flight together
  constexpr int CB = W4 ? 1 : 2;  // 16-byte chunks of a W row per lane and step
  // k of a lane's two operands within a step: 16 q and 64 + 16 q (a load instruction covers 64 contiguous
  // bytes of each row), or, next to packed weights whose 16 bytes hold 32 k, 32 q and 32 q + 16
  constexpr int QA = W4 ? 32 : 16, HA = W4 ? 16 : 64;
  __shared__ v4i red[NW][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int r = lane & 15, q = lane >> 4;
  const int64_t m0 = (int64_t)blockIdx.y * 16, n0 = (int64_t)blockIdx.x * 16;
  const int kb_a = (int)K, kb_w = W4 ? (int)(K >> 1) : (int)K;  // bytes per row
  // rows past the edge re-read the last row; never stored
  const int64_t ra = m0 + r < M ? m0 + r : M - 1, rw = n0 + r < N ? n0 + r : N - 1;
  const uint8_t* pa = reinterpret_cast<const uint8_t*>(A) + ra * kb_a;
  const uint8_t* pw = reinterpret_cast<const uint8_t*>(Wv) + rw * kb_w;
  v4i acc = v4i{0, 0, 0, 0};

  const int steps = (int)((K + 127) >> 7);
  for (int s0 = wave; s0 < steps; s0 += NW * U) {
    v4i a[U][2], b[U][CB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = s0 + u * NW;
      if (s < steps) {  // wave-uniform
        const int ka = s * 128 + q * QA, kw = W4 ? ka >> 1 : ka;
        a[u][0] = load_chunk16(pa, kb_a, ka);
        a[u][1] = load_chunk16(pa, kb_a, ka + HA);
#pragma unroll
        for (int c = 0; c < CB; ++c) b[u][c] = load_chunk16(pw, kb_w, kw + HA * c);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = s0 + u * NW;
      if (s < steps) {
        const int ka = s * 128 + q * QA, kw = W4 ? ka >> 1 : ka;
        if (s == steps - 1) {  // the step that may reach past the row's end
          a[u][0] = fix_chunk16(a[u][0], kb_a, ka);
          a[u][1] = fix_chunk16(a[u][1], kb_a, ka + HA);
#pragma unroll
          for (int c = 0; c < CB; ++c) b[u][c] = fix_chunk16(b[u][c], kb_w, kw + HA * c);
        }
        v4i bw[2] = {b[u][0], b[u][CB - 1]};
        if constexpr (W4) {  // 32 nibbles -> 32 bytes n << 4, in k order
          unsigned e[8];
          expand8((unsigned)b[u][0].x, e[0], e[1]);
          expand8((unsigned)b[u][0].y, e[2], e[3]);
          expand8((unsigned)b[u][0].z, e[4], e[5]);
          expand8((unsigned)b[u][0].w, e[6], e[7]);
          bw[0] = v4i{(int)e[0], (int)e[1], (int)e[2], (int)e[3]};
          bw[1] = v4i{(int)e[4], (int)e[5], (int)e[6], (int)e[7]};
        }
        // W as the row operand: a lane then holds four consecutive n of one output row
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(bw[0], a[u][0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(bw[1], a[u][1], acc, 0, 0, 0);
      }
    }
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave > 0) return;

  // lane (r, q) of the first wave finishes outputs n .. n + 3 of row m
  v4i s = red[0][lane];
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    const v4i o = red[w][lane];
    s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
  }
  const int64_t m = m0 + r, n = n0 + 4 * q;
  const bool want_y = Y || epi.amax || epi.codes;
  float amax = 0.0f;
  if (m < M && n < N) {
    int a[4] = {s.x, s.y, s.z, s.w};
    float y[4], code[4];
    const float sa = want_y ? a_scale[0] : 0.0f;
    float q_scale, q_inv = 0.0f, q_max = 0.0f;
    if (epi.codes) {
      bit_constants(epi.q_absmax[0], epi.q_bits, q_scale, q_inv);
      q_max = (float)((1 << (epi.q_bits - 1)) - 1);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (W4) a[e] >>= 4;  // exact: every product carried the factor 16
      const bool in = n + e < N;
      const float sw = want_y ? w_scale[w_per_row ? (in ? n + e : n) : 0] : 0.0f;
      y[e] = apply_act(((float)a[e] * sa) * sw, epi.act);
      if (in) amax = fmaxf(amax, fabsf(y[e]));
      code[e] = code_f(y[e], q_inv, q_max);
    }
    if (vec) {  // N % 4 == 0 and aligned outputs: the four n are all in range
      if (ACC) *reinterpret_cast<v4i*>(ACC + m * N + n) = v4i{a[0], a[1], a[2], a[3]};
      if (Y) *reinterpret_cast<float4*>(Y + m * N + n) = make_float4(y[0], y[1], y[2], y[3]);
      if (epi.codes)
        *reinterpret_cast<unsigned*>(epi.codes + m * N + n) =
            ((unsigned)(int)code[0] & 0xFFu) | (((unsigned)(int)code[1] & 0xFFu) << 8) |
            (((unsigned)(int)code[2] & 0xFFu) << 16) | ((unsigned)(int)code[3] << 24);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (n + e >= N) break;
        if (ACC) ACC[m * N + n + e] = a[e];
        if (Y) Y[m * N + n + e] = y[e];
        if (epi.codes) epi.codes[m * N + n + e] = (int8_t)(int)code[e];
      }
    }
  }
  if (epi.amax) {
    const float w = wave_max(amax);
    if (lane == 0) atomicMax(epi.amax, abs_key(w));
  }
}

// Measured (us, this kernel with 4 | 8 waves against the tiled kernels, int8, one 16 x 16 tile per CU at
// most): K = 256 3.0 | 3.1 / 3.9, 1024 3.7 | 3.7 / 6.5, 2304 4.9 | 4.7 / 7.8, 4608 7.2 | 6.7 / 8.7, the same for
// packed int4.  Two tiles per CU (256 x 512): K = 256 3.2 | 5.0 / 4.1, 1024 4.6 | 6.2 / 7.3, 2304 7.1 | 8.4 / 8.3,
// but 4608 11.4 | 12.6 / 10.1; from four tiles per CU on the tiled kernels win at every K (384 x 768: 6.1 / 4.1,
// 9.2 / 6.6, 15.0 / 7.9).
// amax: with a running maximum, where the fast tiled kernels could take over, only up to one tile per CU: the atomics on its one address queue up (with ReLU and its
// maximum 128 x 768 x 768 9.5 us against 7.4, 256 x 2304 x 512 14.3 against 10.4).
int skinny_waves(int64_t M, int64_t N, int64_t K, bool amax) {
  const int64_t tm = (M + 15) / 16, tn = (N + 15) / 16;
  if (tm > 2 * kNumCU || tn > 2 * kNumCU || (amax && tm * tn > kNumCU)) return 0;
  if (tm * tn <= kNumCU) return K >= 2048 ? 8 : 4;
  return tm * tn <= 2 * kNumCU && K <= 2304 ? 4 : 0;
}

int launch_skinny(int waves, bool w4, const DmaArgs& d) {
  const dim3 grid((unsigned)((d.N + 15) / 16), (unsigned)((d.M + 15) / 16));
  const int vec = (d.N & 3) == 0 && (!d.y_out || aligned16(d.y_out)) && (!d.acc_out || aligned16(d.acc_out)) &&
                  (!d.epi.codes || (reinterpret_cast<uintptr_t>(d.epi.codes) & 3u) == 0);
#define MPQ_SK(NW_, W4_)                                                                                         \
  qgemm_skinny<NW_, W4_><<<grid, NW_ * 64, 0, d.st>>>(d.a_q, d.w_q, d.M, d.N, d.K, d.a_scale, d.w_scale, d.per_row, \
                                                      d.y_out, d.acc_out, d.epi, vec)
  if (waves == 8) {
    if (w4) MPQ_SK(8, true);
    else MPQ_SK(8, false);
  } else {
    if (w4) MPQ_SK(4, true);
    else MPQ_SK(4, false);
  }
#undef MPQ_SK
  return launch_status();
}

}  // namespace mpq
