// hutchinson.hip -- Hutchinson's estimate of the trace of the Hessian (paper Sec. 3.2.3,
// E_Hessian = E[Tr(d^2 L / d w_i^2)]) for the one case that needs no network behind it: a linear
// layer Y = X W' under L = mean((Y - T)^2).  L is quadratic in W with Hessian
// (2 / (M N)) (I_N (x) X'X), so a probe's quadratic form is a sum of ||X v||^2 over K-vectors v,
// and Tr(H) ~= (2 / M) mean_p ||X v_p||^2 (exact value: (2 / M) ||X||_F^2).
//
//   mpq_rademacher       the probes: random signs, one Philox bit per element
//   mpq_hutchinson_quad  quad[p] = ||X v_p||^2 = sum_m (sum_k X[m][k] v[p][k])^2
//   mpq_hutchinson_quad_signs  the same with the sign probes drawn inside the kernel (the bits
//                        mpq_rademacher would store): no probe matrix is read at all
//
// The second is a dense contraction X [M x K] times V' [K x P] followed by a column-wise sum of
// squares, so it runs on the matrix cores: the third on the bf16 ones (products with signs are exact
// there too, see hutch_signs_k), the second on the fp32 matrix cores (v_mfma_f32_32x32x2_f32; products with +-1 are
// exact, the sums over k round in fp32).  X is read once per group of up to 64 probes; with 32
// probes the kernel is bound by that read (4 bytes per element of X against 64 flops), with 64
// the fp32 matrix rate is level with it.  V (P x K floats, at most a few MB) stays in L2.
//
// A workgroup of eight waves owns 32 rows of X at a time; the waves split k between them (a
// contiguous eighth each) and walk it in chunks of 32 (lane l: row l % 32, sixteen consecutive k in
// half l / 32 of the chunk, loaded as four 16-byte pieces that feed four K = 2 matrix steps each), add their 32 x 32 partial products
// through LDS, and wave 0 squares and accumulates.  Lane l of a product tile holds column
// p = l % 32 and sixteen of the rows m, so the column sums of squares need no cross-lane work
// until the very end.
#include "common.hpp"
#include "philox.hpp"

#include <atomic>

namespace mpq {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kHW = 8;           // waves per workgroup; they split k
constexpr int kProbeGroup = 64;  // probes per pass over X: the width at which the fp32 matrix rate
                                 // (64 flops per byte of X at the HBM rate) and the read of X balance

// thread w owns word w of the sign stream: elements 32 w .. 32 w + 31
__global__ __launch_bounds__(kBlock) void rademacher_k(unsigned long long seed, unsigned long long sid,
                                                       int64_t n, float* __restrict__ out) {
  const int64_t w = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t e0 = w << 5;
  if (e0 >= n) return;
  const unsigned long long g = (unsigned long long)(w >> 2);
  const U4 r = philox4x32_10((unsigned)g, (unsigned)(g >> 32), (unsigned)sid, (unsigned)(sid >> 32),
                             (unsigned)seed, (unsigned)(seed >> 32) ^ 0x5241444Du);
  const unsigned sel = (unsigned)w & 3u;
  const unsigned word = sel == 0 ? r.a : sel == 1 ? r.b : sel == 2 ? r.c : r.d;
#pragma unroll 8
  for (int t = 0; t < 32; ++t)
    if (e0 + t < n) out[e0 + t] = ((word >> t) & 1u) ? -1.0f : 1.0f;
}

// four floats at p (k .. k+3) with everything at or past `left` elements zeroed
template <bool VEC>
__device__ __forceinline__ float4 load4f(const float* __restrict__ p, int64_t left, bool ok) {
  if (VEC) {  // left is a multiple of 4: the piece is whole or absent
    return (ok && left > 0) ? *reinterpret_cast<const float4*>(p) : make_float4(0.f, 0.f, 0.f, 0.f);
  } else {
    float4 r;
    r.x = (ok && left > 0) ? p[0] : 0.f;
    r.y = (ok && left > 1) ? p[1] : 0.f;
    r.z = (ok && left > 2) ? p[2] : 0.f;
    r.w = (ok && left > 3) ? p[3] : 0.f;
    return r;
  }
}

// One chunk of a wave's operands: CH pieces of four k each of X row `row` and of PB x 32 probe
// rows (lane (row, half) owns the k range [c * 8 CH + half * 4 CH, + 4 CH) of chunk c).
template <int PB, int CH>
struct Operands {
  float4 x[CH];
  float4 v[PB][CH];
};

// piece e (four k) of the chunk that starts at kb for this lane
template <int PB, int CH, bool VEC>
__device__ __forceinline__ void load_piece(Operands<PB, CH>& o, int e, const float* __restrict__ xr, bool m_ok,
                                           const float* __restrict__ V, int64_t P, int64_t K, int64_t kb, int row,
                                           bool live) {
  const int64_t k = kb + 4 * e;
  o.x[e] = load4f<VEC>(xr + k, K - k, live && m_ok);
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    const int64_t p = pb * 32 + row;
    const bool p_ok = live && p < P;
    o.v[pb][e] = load4f<VEC>(V + (p_ok ? p : 0) * K + k, K - k, p_ok);
  }
}

// part: float [gridDim.x][PB * 32], this workgroup's share of sum_m (X V')[m][p]^2
template <int PB, bool VEC>
__global__ __launch_bounds__(kHW * 64, 4) void hutch_k(const float* __restrict__ X, int64_t M, int64_t K,
                                                       const float* __restrict__ V, int64_t P,
                                                       float* __restrict__ part) {
  constexpr int CH = 4;               // pieces per chunk and lane
  constexpr int CK = 8 * CH;          // k per chunk
  __shared__ float red[kHW - 1][PB][16][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int row = lane & 31, half = lane >> 5;
  const int64_t nchunk = (K + CK - 1) / CK;
  const int64_t nblk = (M + 31) >> 5;
  // wave w takes the chunks [c_lo, c_hi): a contiguous share of k
  const int64_t per = (nchunk + kHW - 1) / kHW;
  const int64_t c_lo = wave * per;
  const int64_t c_hi = c_lo + per < nchunk ? c_lo + per : nchunk;
  float s[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) s[pb] = 0.0f;

  for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const int64_t m = blk * 32 + row;
    const bool m_ok = m < M;
    const float* xr = X + (m_ok ? m : 0) * K;
    v16f acc[PB];
#pragma unroll
    for (int pb = 0; pb < PB; ++pb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[pb][v] = 0.0f;

    // A piece's registers are refilled with the same piece of the wave's next chunk as soon as
    // the matrix steps that read them have been issued: loads run most of a chunk ahead of their
    // use without a second set of registers.
    Operands<PB, CH> o;
#pragma unroll
    for (int e = 0; e < CH; ++e)
      load_piece<PB, CH, VEC>(o, e, xr, m_ok, V, P, K, c_lo * CK + half * (CK / 2), row, c_lo < c_hi);
    for (int64_t c = c_lo; c < c_hi; ++c) {
      const int64_t kn = (c + 1) * CK + half * (CK / 2);
      const bool more = c + 1 < c_hi;
#pragma unroll
      for (int e = 0; e < CH; ++e) {
        float4 v[PB];
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) v[pb] = o.v[pb][e];
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) acc[pb] = __builtin_amdgcn_mfma_f32_32x32x2f32(o.x[e].x, v[pb].x, acc[pb], 0, 0, 0);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) acc[pb] = __builtin_amdgcn_mfma_f32_32x32x2f32(o.x[e].y, v[pb].y, acc[pb], 0, 0, 0);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) acc[pb] = __builtin_amdgcn_mfma_f32_32x32x2f32(o.x[e].z, v[pb].z, acc[pb], 0, 0, 0);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) acc[pb] = __builtin_amdgcn_mfma_f32_32x32x2f32(o.x[e].w, v[pb].w, acc[pb], 0, 0, 0);
        load_piece<PB, CH, VEC>(o, e, xr, m_ok, V, P, K, kn, row, more);
      }
    }

    // the k shares of the 32 x 32 products meet in wave 0, in a fixed order
    if (wave > 0) {
#pragma unroll
      for (int pb = 0; pb < PB; ++pb)
#pragma unroll
        for (int v = 0; v < 16; ++v) red[wave - 1][pb][v][lane] = acc[pb][v];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int pb = 0; pb < PB; ++pb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          float d = acc[pb][v];
#pragma unroll
          for (int w = 0; w < kHW - 1; ++w) d += red[w][pb][v][lane];
          s[pb] = __builtin_fmaf(d, d, s[pb]);
        }
    }
    __syncthreads();  // red is free again
  }
  if (wave == 0) {
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      const float t = s[pb] + __shfl_xor(s[pb], 32);  // the two halves hold different rows of the same column
      if (lane < 32) part[(int64_t)blockIdx.x * (PB * 32) + pb * 32 + lane] = t;
    }
  }
}

// =====================================================================================================
// The sign probes drawn in the kernel.
//
// Products with +-1 need no fp32 multiplier: x is split exactly into three bf16 numbers (the 24 bits of its
// significand, eight at a time: hi = the top of x, mid = the top of x - hi, lo = the rest; all three
// differences are exact), the signs are bf16, and v_mfma_f32_32x32x16_bf16 adds the exact products in
// fp32.  Three such steps take 96 clocks where sixteen k took 512 on v_mfma_f32_32x32x2_f32, with an eighth
// of the roundings of the sum, so what bounds the kernel is the read of X: 67 M elements x 4 bytes.
//
// X travels global -> LDS in tiles of 32 rows x 32 k by direct loads of whole 128-byte lines (a lane that
// reads its own row, as the operand layout wants it, touches 64 lines per load instruction and keeps the
// memory at 4.4 TB/s), four tiles deep per wave.  Every wave has a ring of its own, so there is no
// barrier in the k loop: a wave waits for its own loads only.  Waves split k in shares of whole 128-k blocks;
// a block is what one Philox call per lane serves (four words, each half of a lane pair takes 16 bits of
// each), or two where K is no multiple of 128 and a probe's blocks straddle Philox blocks.
//
// us with the finishing kernel, fp32 steps against this: 16384 x 4096 32 probes 77 -> 54 (5.0 TB/s), 64 probes
// 110 -> 63; 16384 x 2048 42 -> 28; 70000 x 512 44 -> 31; 9000 x 2064 36 -> 33; 1000 x 4096 30 -> 19; 16384 x 64
// 7.7 -> 7.0.  Below about 100 K elements both are launch and latency: 64 x 512 8.8 -> 7.3, 64 x 64 6.2 -> 5.2, 64 x 128
// 6.3 -> 5.2, 89 x 144 6.75 -> 5.7, 4798 x 192 7.2 -> 6.1.
// =====================================================================================================
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

struct Signs {
  unsigned long long seed, sid, first;  // first: index of probe row 0 of this pass in the sign matrix
};

// the Philox block that holds element `base` of the sign matrix
__device__ __forceinline__ U4 sign_block(const Signs& sg, unsigned long long base) {
  const unsigned long long g = base >> 7;
  return philox4x32_10((unsigned)g, (unsigned)(g >> 32), (unsigned)sg.sid, (unsigned)(sg.sid >> 32),
                       (unsigned)sg.seed, (unsigned)(sg.seed >> 32) ^ 0x5241444Du);
}
// eight signs (bits 0..7 of `bits`) as bf16 +1 / -1, lowest bit first
__device__ __forceinline__ v8bf sign_operand(unsigned bits) {
  unsigned d[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    d[j] = 0x3F803F80u | ((bits << (15 - 2 * j)) & 0x8000u) | ((bits << (30 - 2 * j)) & 0x80000000u);
  return __builtin_bit_cast(v8bf, d);
}

// x = hi + mid + lo, exactly, for eight x
__device__ __forceinline__ void split3(const float (&x)[8], v8bf& hi, v8bf& mid, v8bf& lo) {
  unsigned h[4], m[4], l[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float a = x[2 * j], b = x[2 * j + 1];
    const unsigned ua = (unsigned)bits_from_f(a), ub = (unsigned)bits_from_f(b);
    h[j] = __builtin_amdgcn_perm(ub, ua, 0x07060302u);
    const float ra = a - f_from_bits((int)(ua & 0xFFFF0000u)), rb = b - f_from_bits((int)(ub & 0xFFFF0000u));
    const unsigned va = (unsigned)bits_from_f(ra), vb = (unsigned)bits_from_f(rb);
    m[j] = __builtin_amdgcn_perm(vb, va, 0x07060302u);
    const float la = ra - f_from_bits((int)(va & 0xFFFF0000u)), lb = rb - f_from_bits((int)(vb & 0xFFFF0000u));
    l[j] = __builtin_amdgcn_perm((unsigned)bits_from_f(lb), (unsigned)bits_from_f(la), 0x07060302u);
  }
  hi = __builtin_bit_cast(v8bf, h);
  mid = __builtin_bit_cast(v8bf, m);
  lo = __builtin_bit_cast(v8bf, l);
}

constexpr int kSW = 8;                   // most waves of a workgroup
constexpr int kRing = 4;                 // tiles of a wave's ring
constexpr int kTileBytes = 32 * 128;     // 32 rows x 32 floats
// LDS of a workgroup of ks * groups waves: the rings, and the partial products of all but the first wave of a
// group or, in their place, the last step's sums
constexpr int signs_lds(int ks, int groups, int ring = kRing) {
  const int shares = (ks - 1) * groups * 16 * 64 * (int)sizeof(float), sums = groups * 2 * 32 * (int)sizeof(double);
  return ks * groups * ring * kTileBytes + (shares > sums ? shares : sums);
}

static __device__ __attribute__((aligned(16))) int g_zeros16[4];  // never written: rows and k past the edge

// ks: waves that split k (1, 2, 4 or 8); the workgroup's ks * groups waves work on `groups` blocks of 32 rows
// at a time
// ONE: K <= 256, a single trip, a wave for each 32 k; its ring is one tile
// part: the sums of squares of 32 rows are fp32, everything above them is double: with per_block float
// [row blocks][PB * 32], one such sum each (what the workspace has room for up to kBlockSums of them), else
// float [gridDim.x][2][PB * 32], the workgroup's share as the nearest float and what is left of it
template <int PB, bool ONE>
__global__ __launch_bounds__(kSW * 64) void hutch_signs_k(const float* __restrict__ X, int64_t M, int64_t K,
                                                          Signs sg, int ks, int groups, int iters, int per_block,
                                                          float* __restrict__ part) {
  constexpr int RING = ONE ? 1 : kRing;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  float* red = reinterpret_cast<float*>(lds + ks * groups * RING * kTileBytes);  // [(ks - 1) * groups][16][64]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int row = lane & 31, half = lane >> 5;
  const int group = wave / ks, kshare = wave % ks;
  const int64_t nblock = (K + 127) >> 7;                // 128-k blocks
  const int64_t per = ONE ? 1 : (nblock + ks - 1) / ks;  // of a wave: kshare, kshare + ks, ...; those past K read zeros
  const unsigned ring = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)lds + (unsigned)(wave * RING * kTileBytes);
  const char* my = lds + wave * RING * kTileBytes;
  const char* zero = reinterpret_cast<const char*>(g_zeros16);

  // Requests run kRing tiles ahead of the work, across row blocks.  Load i of a tile brings rows
  // 8 i .. 8 i + 7: lane l row 8 i + l / 8, and to keep the operand reads free of bank conflicts slot s of
  // row r holds the 16-byte chunk s ^ ((r >> 1) & 7) of its 128 bytes.
  // Rows past the edge re-read the last row (their products are dropped below); the lane's four addresses
  // move along with the tiles, so that a request costs two additions per load.
  // Nothing is requested past the last row block: at the end the kernel would wait for it.
  int64_t rq_b = 0;                       // number of the wave's 128-k block
  int64_t rq_left = (int64_t)iters * per;  // blocks still to be requested in whole
  int64_t rq_blk = (int64_t)blockIdx.x * groups + group;
  const char* src[4];
  auto start_block = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int64_t m = rq_blk * 32 + 8 * i + (lane >> 3);
      if (m >= M) m = M - 1;
      const int c = (lane & 7) ^ ((4 * i + (lane >> 4)) & 7);
      src[i] = reinterpret_cast<const char*>(X + m * K + (int64_t)kshare * (ONE ? 32 : 128) + 4 * c);
    }
  };
  start_block();
  const int64_t last_k = K - 32;  // K % 16 == 0 and a chunk of four is whole or absent
  auto request = [&](unsigned slot) {  // tile `slot` of the block
    if (rq_left == 0) return;
    const int64_t k0 = ONE ? kshare * 32 : ((kshare + rq_b * ks) * 4 + (int)slot) * 32;
    const bool edge = k0 > last_k;  // wave-uniform
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const char* p = src[i];
      if (edge && k0 + 4 * (int)((lane & 7) ^ ((4 * i + (lane >> 4)) & 7)) >= K) p = zero;
      // M0 holds the LDS address of lane 0; the wait state is the one the ISA asks for after its write
      asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(p),
                   "s"(ring + slot * kTileBytes + i * 1024u)
                   : "memory");
      src[i] += 128;
    }
    if (slot == RING - 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i) src[i] += (ks - 1) * 512;
      --rq_left;
      if (++rq_b == per) {
        rq_b = 0;
        rq_blk += (int64_t)gridDim.x * groups;
        start_block();
      }
    }
  };
  static_assert(kRing == 4, "tile t of a 128-k block lives in ring slot t");
  // (a wave whose only block is cut off by K requests and multiplies the tiles in front of K alone: there the
  // kernel is latency from end to end)
  const int cut = ONE ? 1 : rq_left == 1 && K < ((int64_t)kshare + 1) * 128 ? (int)((K - (int64_t)kshare * 128 + 31) >> 5) : 4;
#pragma unroll 1
  for (int t = 0; t < cut; ++t) request((unsigned)t);
  if (cut < 4) rq_left = 0;

  double sum[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) sum[pb] = 0.0;
  const bool whole_blocks = (K & 127) == 0;
  const unsigned sw = (unsigned)(row >> 1) & 7u;
  // the lane's four chunks of a tile: k = 16 half + 4 e
  unsigned off[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) off[e] = (unsigned)row * 128u + ((((unsigned)half * 4u + e) ^ sw) << 4);

  for (int it = 0; it < iters; ++it) {
    v16f acc[PB];
#pragma unroll
    for (int pb = 0; pb < PB; ++pb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[pb][v] = 0.0f;
    for (int64_t b = ONE ? kshare >> 2 : kshare, b_end = ONE ? b + 1 : per * ks; b < b_end; b += ks) {
      U4 words[PB];
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        const unsigned long long base = (sg.first + (unsigned long long)(pb * 32 + row)) * (unsigned long long)K +
                                        (unsigned long long)b * 128u;
        if (whole_blocks) {
          words[pb] = sign_block(sg, base);
        } else {  // the 128 signs start at any multiple of 16 elements: cut out of two blocks, in named values (an
          // array of words went to scratch memory: 4798 x 192 7.8 us against 7.15)
          const U4 p0 = sign_block(sg, base), p1 = sign_block(sg, base + 128u);
          const unsigned at = (unsigned)base & 127u;
          auto cut2 = [&](unsigned lo, unsigned hi) { return (at & 16u) ? (lo >> 16) | (hi << 16) : lo; };
          const unsigned w0 = cut2(p0.a, p0.b), w1 = cut2(p0.b, p0.c), w2 = cut2(p0.c, p0.d), w3 = cut2(p0.d, p1.a),
                         w4 = cut2(p1.a, p1.b), w5 = cut2(p1.b, p1.c), w6 = cut2(p1.c, p1.d);
          const bool one = at & 32u, two = at & 64u;
          const unsigned u0 = one ? w1 : w0, u1 = one ? w2 : w1, u2 = one ? w3 : w2, u3 = one ? w4 : w3, u4 = one ? w5 : w4,
                         u5 = one ? w6 : w5;
          words[pb] = two ? U4{u2, u3, u4, u5} : U4{u0, u1, u2, u3};
        }
        if (ONE)
          words[pb].a = (kshare & 2) ? ((kshare & 1) ? words[pb].d : words[pb].c) : (kshare & 1) ? words[pb].b : words[pb].a;
      }
#pragma unroll 1
      for (int t = 0; t < cut; ++t) {  // tile t of the block sits in ring slot t (rolled: the code is fetched cold)
        // all but the youngest three tiles; in the wave's last block no younger ones follow
        if (rq_left > 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kRing - 1) * 4) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        float x[2][8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float4 v = *reinterpret_cast<const float4*>(my + t * kTileBytes + off[e]);
          x[e >> 1][(e & 1) * 4 + 0] = v.x;
          x[e >> 1][(e & 1) * 4 + 1] = v.y;
          x[e >> 1][(e & 1) * 4 + 2] = v.z;
          x[e >> 1][(e & 1) * 4 + 3] = v.w;
        }
        // the tile is in registers: its slot can be filled again
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        request((unsigned)t);
#pragma unroll
        for (int st = 0; st < 2; ++st) {
          v8bf hi, mid, lo;
          split3(x[st], hi, mid, lo);
#pragma unroll
          for (int pb = 0; pb < PB; ++pb) {
            const v8bf v = sign_operand((half ? words[pb].a >> 16 : words[pb].a) >> (8 * st));
            acc[pb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo, v, acc[pb], 0, 0, 0);
            acc[pb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mid, v, acc[pb], 0, 0, 0);
            acc[pb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi, v, acc[pb], 0, 0, 0);
          }
        }
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) words[pb] = U4{words[pb].b, words[pb].c, words[pb].d, 0u};
      }
    }
    // the k shares of a row block's 32 x 32 products meet in its first wave, in a fixed order
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      float* mine = red + (int64_t)(group * (ks - 1) + kshare - 1) * (16 * 64) + lane;
      if (kshare > 0) {
#pragma unroll
        for (int v = 0; v < 16; ++v) mine[v * 64] = acc[pb][v];
      }
      __syncthreads();
      if (kshare == 0) {
        // the lane's row of register v is m_lo + 8 (v / 4) + v % 4
        const int64_t block = ((int64_t)it * gridDim.x + blockIdx.x) * groups + group;
        const int64_t m_lo = block * 32 + 4 * half;
        const float* others = red + (int64_t)group * (ks - 1) * (16 * 64) + lane;
        for (int w = 0; w < ks - 1; ++w)  // sixteen independent reads per share
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[pb][v] += others[(w * 16 + v) * 64];
        float s = 0.0f;
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (m_lo + (v >> 2) * 8 + (v & 3) < M) s = __builtin_fmaf(acc[pb][v], acc[pb][v], s);
        if (per_block) {
          s += __shfl_xor(s, 32);  // the two halves hold different rows of the same column
          if (lane < 32 && block * 32 < M) part[block * (PB * 32) + pb * 32 + lane] = s;
        } else {
          sum[pb] += (double)s;
        }
      }
      __syncthreads();  // red is free again
    }
  }
  if (per_block) return;  // uniform over the grid; no request is in flight
  double* sums = reinterpret_cast<double*>(red);
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    const double t = sum[pb] + __shfl_xor(sum[pb], 32);
    if (kshare == 0 && lane < 32) sums[(group * PB + pb) * 32 + lane] = t;
  }
  __syncthreads();
  if ((int)threadIdx.x < PB * 32) {
    double t = 0.0;
    for (int g = 0; g < groups; ++g) t += sums[g * PB * 32 + threadIdx.x];
    float* dst = part + (int64_t)blockIdx.x * 2 * (PB * 32) + threadIdx.x;
    dst[0] = (float)t;
    dst[PB * 32] = (float)(t - (double)(float)t);
  }
}

// quad[p] = sum over workgroups of part[b][p], in double, fixed order; one workgroup per probe
__global__ __launch_bounds__(kBlock) void hutch_finish(const float* __restrict__ part, int nblocks, int width,
                                                       double* __restrict__ quad) {
  const int p = blockIdx.x;
  double t = 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < nblocks; b += kBlock) t += (double)part[(int64_t)b * width + p];
  t = wave_sum(t);
  __shared__ double sm[kBlock / kWave];
  if ((threadIdx.x & (kWave - 1)) == 0) sm[threadIdx.x / kWave] = t;
  __syncthreads();
  if (threadIdx.x == 0) quad[p] = (sm[0] + sm[1]) + (sm[2] + sm[3]);
}

static int probe_blocks(int64_t pg) { return pg <= 32 ? 1 : 2; }

constexpr int64_t kBlockSums = (int64_t)kNumCU * 4;

// workgroups of one pass: a few per CU, every lane accumulating at most 256 row blocks in fp32
static int64_t hutch_grid(int64_t M, int pb) {
  const int64_t nblk = (M + 31) >> 5;
  (void)pb;
  int64_t g = kBlockSums;
  if (g > nblk) g = nblk;
  const int64_t need = (nblk + 255) / 256;
  return g > need ? g : need;
}

// How a pass is laid out: ks waves per row block, `groups` row blocks per workgroup, `grid` workgroups
// (one per CU at a time, what the LDS allows) that make `iters` trips.
// The workspace holds hutch_grid rows of 64 floats: up to kBlockSums row blocks it has one for each of them, above
// that at least kBlockSums, two for each of the kNumCU workgroups.
// The layout with the least estimated time is taken: a trip costs the 128-k blocks of a wave times what one
// takes, 1.4 us (its own latencies) plus 0.7 us for every wave of the CU (the memory rate they share) -- from
// 16384 x 4096 in four and in eight waves per CU, 67 and 55 us -- and 1 us for adding the shares.
struct SignsPlan {
  int ks = 1, groups = 1, iters = 1;
  bool one = false;  // a tile of 32 k per wave
  int64_t grid = 1;
};
static SignsPlan plan_signs(int64_t M, int64_t K) {
  const int64_t nblk = (M + 31) >> 5, nb = (K + 127) >> 7;
  SignsPlan best;
  // Up to two blocks of k are latency from end to end, a block's four tiles one after the other in a wave: with a wave
  // each 64 x 128 6.75 -> 5.25 us, 4000 x 128 (40 probes) 8.35 -> 6.65, 64 x 64 5.75 -> 5.2, 1000 x 192 7.0 -> 5.9,
  // 8192 x 256 (40 probes) 9.05 -> 8.4, and the fp32 chains are shorter: 89 x 144 rms error 4.6e-8 -> 3.8e-8.
  if (nb <= 2 && nblk <= kNumCU) {
    best.ks = (int)((K + 31) >> 5);
    best.grid = nblk;
    best.one = true;
    return best;
  }
  double least = 0.0;
  for (int ks = 1; ks <= kSW; ks *= 2)
    for (int groups = 1; groups * ks <= kSW; groups *= 2) {
      SignsPlan p;
      p.ks = ks;
      p.groups = groups;
      const int64_t items = (nblk + groups - 1) / groups;
      p.grid = items < kNumCU ? items : kNumCU;
      p.iters = (int)((items + p.grid - 1) / p.grid);
      const double per = (double)((nb + ks - 1) / ks);
      const double cost = p.iters * (per * (1.4 + 0.7 * ks * groups) + 1.0);
      if (least == 0.0 || cost < least) {
        least = cost;
        best = p;
      }
    }
  return best;
}

// Dynamic LDS above 64 KiB has to be allowed once per kernel and device.
static int signs_allow_lds() {
  static std::atomic<unsigned> done[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (done[dev].load(std::memory_order_relaxed)) return MPQ_OK;
  for (const void* k : {reinterpret_cast<const void*>(&hutch_signs_k<1, false>), reinterpret_cast<const void*>(&hutch_signs_k<2, false>)}) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, signs_lds(kSW, 1));
    if (e != hipSuccess) { set_last_hip_error((int)e); return MPQ_ERR_HIP; }
  }
  done[dev].store(1, std::memory_order_relaxed);
  return MPQ_OK;
}

}  // namespace mpq

using namespace mpq;

namespace mpq {
int prepare_hutchinson() { return signs_allow_lds(); }
}  // namespace mpq

extern "C" int mpq_rademacher(uint64_t seed, uint64_t stream_id, int64_t rows, int64_t cols, float* v_out,
                              void* stream) {
  if (!v_out) return MPQ_ERR_NULL;
  if (rows <= 0 || cols <= 0 || mul_overflows(rows, cols) || rows * cols > ((int64_t)1 << 38)) return MPQ_ERR_SHAPE;
  const int64_t n = rows * cols;
  const int64_t words = (n + 31) >> 5;
  rademacher_k<<<(unsigned)((words + kBlock - 1) / kBlock), kBlock, 0, (hipStream_t)stream>>>(seed, stream_id, n, v_out);
  return launch_status();
}

extern "C" size_t mpq_hutchinson_quad_workspace_bytes(int64_t M, int64_t K, int64_t P) {
  if (M <= 0 || K <= 0 || P <= 0 || mul_overflows(M, K) || mul_overflows(P, K)) return 0;
  size_t most = 0;
  for (int pb = 1; pb <= 2; pb *= 2) {
    const size_t b = (size_t)hutch_grid(M, pb) * (size_t)(pb * 32) * sizeof(float);
    if (b > most) most = b;
  }
  return most;
}

// one pass per group of kProbeGroup probes; v == nullptr draws the signs in the kernel
static int run_hutchinson(const float* x, int64_t M, int64_t K, const float* v, uint64_t seed, uint64_t stream_id,
                          int64_t P, double* quad_out, float* part, hipStream_t st) {
  const bool signs = v == nullptr;
  if (signs) {
    const int rc = signs_allow_lds();
    if (rc != MPQ_OK) return rc;
  }
  const bool vec = !signs && aligned16(x) && aligned16(v) && (K & 3) == 0;
  for (int64_t p0 = 0; p0 < P; p0 += kProbeGroup) {
    const int64_t pg = P - p0 < kProbeGroup ? P - p0 : kProbeGroup;
    const int pb = probe_blocks(pg);
    int64_t sums;  // rows of part
    if (signs) {
      const SignsPlan pl = plan_signs(M, K);
      const int64_t nblk = (M + 31) >> 5;
      const int per_block = nblk <= kBlockSums;
      sums = per_block ? nblk : 2 * pl.grid;
      const Signs sg = {seed, stream_id, (unsigned long long)p0};
      const unsigned g = (unsigned)pl.grid;
      const int threads = pl.ks * pl.groups * 64, lds = signs_lds(pl.ks, pl.groups, pl.one ? 1 : kRing);
#define MPQ_SIGNS(PB_, ONE_) \
  hutch_signs_k<PB_, ONE_><<<g, threads, lds, st>>>(x, M, K, sg, pl.ks, pl.groups, pl.iters, per_block, part)
      if (pl.one && pb == 1) MPQ_SIGNS(1, true);
      else if (pl.one) MPQ_SIGNS(2, true);
      else if (pb == 1) MPQ_SIGNS(1, false);
      else MPQ_SIGNS(2, false);
#undef MPQ_SIGNS
    } else {
      const unsigned g = (unsigned)hutch_grid(M, pb);
      sums = g;
      const float* vp = v + p0 * K;
#define MPQ_HUTCH(PB_)                                                                     \
  (vec ? hutch_k<PB_, true><<<g, kHW * 64, 0, st>>>(x, M, K, vp, pg, part)                 \
       : hutch_k<PB_, false><<<g, kHW * 64, 0, st>>>(x, M, K, vp, pg, part))
      if (pb == 1) MPQ_HUTCH(1);
      else MPQ_HUTCH(2);
#undef MPQ_HUTCH
    }
    hutch_finish<<<(unsigned)pg, kBlock, 0, st>>>(part, (int)sums, pb * 32, quad_out + p0);
  }
  return launch_status();
}

static int check_hutchinson(const float* x, int64_t M, int64_t K, int64_t P, double* quad_out, void* ws,
                            size_t ws_bytes) {
  if (!x || !quad_out) return MPQ_ERR_NULL;
  if (M <= 0 || K <= 0 || P <= 0 || M >= ((int64_t)1 << 31) || P > ((int64_t)1 << 20)) return MPQ_ERR_SHAPE;
  if (mul_overflows(M, K) || mul_overflows(P, K)) return MPQ_ERR_SHAPE;
  if ((reinterpret_cast<uintptr_t>(x) & 3u) || (reinterpret_cast<uintptr_t>(quad_out) & 7u)) return MPQ_ERR_ALIGN;
  if (!ws || ws_bytes < mpq_hutchinson_quad_workspace_bytes(M, K, P)) return MPQ_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(ws) & 3u) return MPQ_ERR_ALIGN;
  return MPQ_OK;
}

extern "C" int mpq_hutchinson_quad(const float* x, int64_t M, int64_t K, const float* v, int64_t P,
                                   double* quad_out, void* ws, size_t ws_bytes, void* stream) {
  if (!v) return MPQ_ERR_NULL;
  if (reinterpret_cast<uintptr_t>(v) & 3u) return MPQ_ERR_ALIGN;
  const int rc = check_hutchinson(x, M, K, P, quad_out, ws, ws_bytes);
  if (rc != MPQ_OK) return rc;
  return run_hutchinson(x, M, K, v, 0, 0, P, quad_out, reinterpret_cast<float*>(ws), (hipStream_t)stream);
}

extern "C" int mpq_hutchinson_quad_signs(const float* x, int64_t M, int64_t K, uint64_t seed, uint64_t stream_id,
                                         int64_t P, double* quad_out, void* ws, size_t ws_bytes, void* stream) {
  const int rc = check_hutchinson(x, M, K, P, quad_out, ws, ws_bytes);
  if (rc != MPQ_OK) return rc;
  if ((K & 15) || !aligned16(x)) return MPQ_ERR_SHAPE;  // a lane's 16 signs of a chunk must sit in one Philox word
  return run_hutchinson(x, M, K, nullptr, seed, stream_id, P, quad_out, reinterpret_cast<float*>(ws),
                        (hipStream_t)stream);
}
