// qgemm_dma.hpp -- the fast path of the quantized linear layer (the evaluation step of the paper's
// Alg. 1 / Alg. 2): the templated multi-stage LDS pipeline fed by direct global->LDS loads, shared by
// the translation units that instantiate one tile size each (qgemm_t*.hip), and the epilogue
// options shared with the generic kernel (qgemm.hip).
#pragma once

#include "common.hpp"

#include <atomic>
#include <type_traits>

namespace mpq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
// the same in memory at any address an element may have
typedef int v4i_any __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u32_any __attribute__((aligned(1)));

// What an epilogue may do beyond Y = (float(acc) * s_A) * s_W[n]:
//  - score: accumulate sum (Y - yref)^2, one double partial per workgroup in `part`;
//  - activation: Y <- act(Y) before it is stored (1 = ReLU, 2 = GELU), and the largest |Y| after
//    the activation merged into amax[0] (an integer atomic max over the bit patterns of the
//    non-negative floats: exact and independent of the order), or one maximum per workgroup in
//    amax_part for a consumer that folds them (256 workgroups that end together wait 2.7 us for
//    each other's atomics on one address);
//  - codes: the activated output quantized on the spot (Eq. 1 with the absmax in q_absmax[0], which
//    an earlier pass over the same product found) and stored as int8 codes, so that the fp32 layer
//    output never travels to HBM and back on its way into the next layer's GEMM.
struct EpiArgs {
  const float* yref;
  double* part;
  int act;
  unsigned* amax;
  const float* q_absmax;
  int q_bits;
  int8_t* codes;
  float* amax_part = nullptr;  // not null: a workgroup leaves its largest |Y| here, at its number, and not in amax
};
constexpr EpiArgs kNoEpi = {nullptr, nullptr, 0, nullptr, nullptr, 0, nullptr};

// GELU(y) = y Phi(y).  The epilogue's arithmetic is not hidden behind anything (every wave of the
// workgroup is in its epilogue at the same time), so Phi is evaluated in about twenty lane
// operations instead of the library erf's fifty: with t = |y|,
//   Phi(-t) = 1/2 erfc(t / sqrt 2) = exp(-t^2 / 2) P(u),  u = 1 / (1 + 0.28 t),
// P a degree-6 polynomial fitted (minimax in the relative error, 4e-7 on 0 <= t <= 6) to
// 1/2 erfcx(t / sqrt 2), and Phi(t) = 1 - Phi(-t).  The form keeps the RELATIVE accuracy in the
// negative tail, where 1 + erf would cancel: in fp32 the result is within 2e-6 relative of the
// exact GELU for y >= -6 (the rounding of t^2 in the exponent dominates) and within 4e-7 |y|
// absolute everywhere (beyond y = -6 GELU itself is below 1e-9 |y|).
__device__ __forceinline__ float gelu_f(float y) {
  const float t = fabsf(y);
  const float u = __builtin_amdgcn_rcpf(__builtin_fmaf(t, 0.28f, 1.0f));
  float p = -0.11208509653806686f;
  p = __builtin_fmaf(p, u, 0.41932520270347595f);
  p = __builtin_fmaf(p, u, -0.29365190863609314f);
  p = __builtin_fmaf(p, u, 0.32605481147766113f);
  p = __builtin_fmaf(p, u, 0.035669293254613876f);
  p = __builtin_fmaf(p, u, 0.12578752636909485f);
  p = __builtin_fmaf(p, u, -0.0010996352648362517f);
  const float tail = __builtin_amdgcn_exp2f((t * t) * -0.72134752044448170f) * p;  // exp(-t^2/2) P(u)
  return y * (y < 0.0f ? tail : 1.0f - tail);
}

__device__ __forceinline__ float apply_act(float y, int act) {
  if (act == 1) return fmaxf(y, 0.0f);
  if (act == 2) return gelu_f(y);
  return y;
}

__device__ __forceinline__ float4 apply_act4(const float4& y, int act) {
  if (act == 1) return make_float4(fmaxf(y.x, 0.0f), fmaxf(y.y, 0.0f), fmaxf(y.z, 0.0f), fmaxf(y.w, 0.0f));
  if (act == 2) return make_float4(gelu_f(y.x), gelu_f(y.y), gelu_f(y.z), gelu_f(y.w));
  return y;
}

// 8 nibbles of `w` (lowest nibble = lowest k) -> 8 bytes, each nibble << 4, in k order
__device__ __forceinline__ void expand8(unsigned w, unsigned& lo, unsigned& hi) {
  const unsigned e = (w << 4) & 0xF0F0F0F0u;  // nibbles 0,2,4,6
  const unsigned o = w & 0xF0F0F0F0u;         // nibbles 1,3,5,7
  lo = __builtin_amdgcn_perm(o, e, 0x05010400u);
  hi = __builtin_amdgcn_perm(o, e, 0x07030602u);
}

// 16 bytes of a row of `row_bytes` bytes from byte k on, at any address (gfx950 loads 16 bytes from any
// byte address; written as a copy so that the compiler knows the pointer is not aligned).  A chunk that
// would pass the row's end is loaded so that it ends there, and fix_chunk16 moves its bytes into place
// and zeroes the rest; chunks wholly past the end come out as zeros.  Rows shorter than 16 bytes are read
// byte by byte.  Nothing outside the row is ever read.
__device__ __forceinline__ v4i load_chunk16(const uint8_t* row, int row_bytes, int k) {
  v4i v;
  if (row_bytes >= 16) {  // uniform over the grid
    const int kk = k <= row_bytes - 16 ? k : row_bytes - 16;
    __builtin_memcpy(&v, row + kk, 16);
  } else {
    unsigned w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < 16; ++b) {
      const unsigned byte = row[k + b < row_bytes ? k + b : row_bytes - 1];
      w[b >> 2] |= (k + b < row_bytes ? byte : 0u) << (8 * (b & 3));
    }
    v = v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
  }
  return v;
}
__device__ __forceinline__ v4i fix_chunk16(const v4i& c, int row_bytes, int k) {
  if (row_bytes < 16) return c;
  const int s = k + 16 - row_bytes;  // bytes the load was moved back by
  if (s <= 0) return c;
  if (s >= 16) return v4i{0, 0, 0, 0};
  uint64_t lo = (uint64_t)(unsigned)c.x | ((uint64_t)(unsigned)c.y << 32);
  uint64_t hi = (uint64_t)(unsigned)c.z | ((uint64_t)(unsigned)c.w << 32);
  if (s >= 8) {
    lo = hi >> (8 * (s - 8));
    hi = 0;
  } else {
    lo = (lo >> (8 * s)) | (hi << (64 - 8 * s));
    hi >>= 8 * s;
  }
  return v4i{(int)(unsigned)lo, (int)(unsigned)(lo >> 32), (int)(unsigned)hi, (int)(unsigned)(hi >> 32)};
}

// =====================================================================================================
// Fast path: multi-stage LDS pipeline fed by direct global->LDS loads (no register staging).
//
// k is walked in tiles of 128 bytes.  One wave-wide global_load_lds_dwordx4 moves 64 x 16 B = 1 KiB
// and the hardware puts lane l's 16 bytes at LDS base + 16 l, so an instruction fills 8 whole tile
// rows (16 rows of a packed-int4 tile).  To get a bank-conflict-free layout anyway, the *global*
// chunk a lane fetches is permuted: LDS slot s of row r holds logical chunk s ^ ((r >> 1) & 7)
// (int8 tiles, 8 chunks per row) or s ^ ((r >> 2) & 3) (packed tiles, 4 chunks per row).  The LDS
// of gfx950 has 64 banks (256 B per clock, measured): a 128-bit operand read is served 16 lanes
// per clock, those lanes read one chunk column of 16 consecutive rows, and with this XOR their
// 16 addresses are distinct modulo 256 B.  The MFMA operand reads apply the same XOR.  Chunks
// beyond K are fetched from a 16-byte block of zeros.
//
// A k tile is requested NSTAGE tiles ahead of the MFMAs that use it, once the stage it goes to has been read for the last
// time; a wave waits only for its own share of the tile it needs next (s_waitcnt vmcnt) and then meets the others at the
// one barrier per k tile (two in qgemm_quad.hpp, which takes the 256 x 256 tile).
//
// What bounds this path: a k tile costs a CU more than either of its halves alone.  On random operands the matrix
// cores sustain 3.6 POP/s in steps of 16x16x64 (3.3 in steps of 32x32x32, which draw more power; constant
// bytes 4.4 and 4.9), so a 128 x 128 x 128 tile is 0.30 us of matrix work on its CU; its 32 KiB come out of the L2 in
// 0.26 us (8 ns per wave-load; 12.5 if a row's share were 64 bytes), its operand reads out of the LDS in 0.19 us, and it
// takes 0.48 us at a clock that falls to 1.8 GHz.  Two to four stages, four or eight waves, k tiles of 128 or 256, two
// barriers per tile instead of one: all within 10 % of each other (4096 x 1024 x 4096, 22.5-25 us).
// =====================================================================================================
#define MPQ_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

static __device__ __attribute__((aligned(16))) int g_zero16[4];  // never written: zero fill for k tails

// The direct-to-LDS load and its wait are written as inline assembly on purpose: when the
// compiler sees the load it cannot tell which LDS bytes are in flight once more than a handful of
// them are outstanding, and puts a full "s_waitcnt vmcnt(0)" in front of every LDS read -- which
// would serialise the pipeline.  Written this way the compiler does not track them, and the
// kernel does the bookkeeping itself: loads return in order, so "vmcnt(n)" means all but the
// youngest n wave-loads of this wave have landed.
// lds_byte_off must be wave-uniform (it travels in M0); lane l's 16 bytes land at +16 l.
// M0 cannot be named as a clobber (the compiler reserves it and rejects it on clobber lists), so the
// kernels that use dma16 must not make the compiler use M0 itself: no dynamically indexed register
// arrays (v_movrel / s_set_gpr_idx), no LDS-direct reads, no GWS or message instructions.  Every
// array in these kernels is indexed at compile time (static_for, #pragma unroll); in the generated
// code of all four tile sizes every reference to M0 is one of the moves below.
__device__ __forceinline__ void dma16(const char* src, unsigned lds_byte_off) {
  // s_nop: the one wait state the ISA asks for between a write of M0 and an LDS-DMA that reads it
  // (the compiler's hazard pass does not look inside inline assembly)
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_byte_off) : "memory");
}
// the same with a wave-uniform base in scalar registers and a 32-bit offset per lane
__device__ __forceinline__ void dma16_base(const char* base, unsigned off, unsigned lds_byte_off) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds_byte_off) : "memory");
}
// one 4-byte value per lane, at +4 l
__device__ __forceinline__ void dma4(const float* src, unsigned lds_byte_off) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "s"(lds_byte_off) : "memory");
}
// One value that is the same for the whole launch and that no kernel in flight writes, by a scalar load wherever it stands.
// Behind an LDS request, which may write anything as far as the compiler knows, an ordinary load becomes a vector
// load, and to wait for that one is to wait for every request in flight: the whole prefetch, where the first barrier needs
// its first k tile (operands in memory, M x K x N, us, ordinary | scalar: 4096 x 1024 x 1024 12.8 | 12.3, 1000 x 2048 x 1000
// 9.8 | 9.3).
__device__ __forceinline__ float load_scalar(const float* p) {
  return *(const __attribute__((address_space(4))) float*)(uintptr_t)p;
}
// The per-channel W scales of a workgroup's columns travel through LDS: the epilogue then needs no global loads between
// its stores.  Every wave fetches them, so that its own wait covers them.  Columns past the edge: any scale.
template <bool VEC>
__device__ __forceinline__ void request_scales(const float* w_scale, int64_t n0, int64_t N, int bn, int lane, unsigned lds_byte_off) {
  if (VEC) {  // N % 4 == 0, w_scale 16-byte aligned
    const int64_t n = n0 + 4 * lane;
    dma16(reinterpret_cast<const char*>(w_scale + (n < N ? n : 0)), lds_byte_off);
  } else {
    for (int i = 0; i < bn; i += 64) {
      const int64_t n = n0 + i + lane;
      dma4(w_scale + (n < N ? n : 0), lds_byte_off + (unsigned)i * 4u);
    }
  }
}
template <int N_>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N_) : "memory");
}
// This wave's LDS reads and writes are done, and so are everyone's.  (__syncthreads would also wait for the stores
// of an epilogue.)
__device__ __forceinline__ void lds_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void meet() {
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// KB: k bytes per stage (128 or 256)
template <int BM, int BN, int WM, int WN, int NSTAGE, bool W4, int KB>
struct DmaCfg {
  static constexpr int DBK = KB;
  static constexpr int CPR = KB / 16;                 // 16-byte chunks per int8 tile row (8 | 16)
  static constexpr int RPI = 64 / CPR;                // tile rows one wave-load covers (8 | 4)
  // swizzle: slot = chunk ^ ((row >> SH) & (CPR-1)); 2^SH rows share 256 bytes (one sweep of the banks)
  static constexpr int SH = CPR == 16 ? 0 : 1;
  static constexpr int PCPR = KB / 32;                // 16-byte chunks per packed-int4 tile row (4 | 8)
  static constexpr int PRPI = 64 / PCPR;              // packed rows per wave-load (16 | 8)
  static constexpr int PSH = PCPR == 8 ? 1 : 2;
  static constexpr int NW = WM * WN;
  static constexpr int NT = NW * 64;
  static constexpr int TM = BM / WM, TN = BN / WN;   // per-wave tile
  static constexpr int FM = TM / 16, FN = TN / 16;   // 16x16 MFMA tiles per wave
  static constexpr int A_STAGE = BM * DBK;
  static constexpr int B_ROW = W4 ? DBK / 2 : DBK;   // bytes of one W tile row in LDS
  static constexpr int B_STAGE = BN * B_ROW;
  static constexpr int STAGE = A_STAGE + B_STAGE;
  static constexpr int SCALE_OFF = NSTAGE * STAGE;    // 1 KiB of per-channel W scales, then the waves' sums
  static constexpr int SUMS_OFF = SCALE_OFF + 1024;
  static constexpr int LDS_BYTES = SCALE_OFF + 2048;
  static constexpr int NLA = BM / RPI;                // wave-loads per A stage
  static constexpr int NLB = W4 ? BN / PRPI : BN / RPI;  // wave-loads per W stage
  static constexpr int LPW = (NLA + NLB) / NW;        // wave-loads per wave per stage
  static_assert(NLA % NW == 0 && NLB % NW == 0, "loads must divide evenly over the waves");
  static_assert(TM % 16 == 0 && TN % 16 == 0, "wave tile is a multiple of 16 x 16");
  static_assert(KB == 256 || KB == 128, "k tile of 128 or 256 bytes");
  static_assert((NSTAGE - 1) * LPW < 64, "vmcnt is a 6-bit counter");
};

// One matrix step into its own accumulator.  Inline assembly, because the compiler is free to give the builtin's
// result another register than the accumulator it came from and does: the 32 accumulators of a wave then
// wander through twice their registers and spill.  What its hazard pass would do is done here: two wait
// states between a vector instruction that writes an operand and the matrix step (zero_acc, expand_half), and
// acc_ready between the last matrix step and the first read of an accumulator.
__device__ __forceinline__ void mma(v4i& acc, const v4i& w, const v4i& a) {
  asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "v"(a));
}
// (The zeros are opaque: a zero vector that the compiler knows lives across the tile loop, spilled by the 256 tile.)
template <int FM, int FN>
__device__ __forceinline__ void zero_acc(v4i (&acc)[FM][FN]) {
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      asm volatile("v_mov_b32 %0, 0\n\tv_mov_b32 %1, 0\n\tv_mov_b32 %2, 0\n\tv_mov_b32 %3, 0"
                   : "=v"(acc[i][j].x), "=v"(acc[i][j].y), "=v"(acc[i][j].z), "=v"(acc[i][j].w));
    }
  asm volatile("s_nop 1" ::: "memory");
}
// The lane's number, formed anew where it is asked for: carried through the k loop of the 256 tile, it and what is derived
// from it (row numbers, addresses of the epilogue) were spilled, as was the zero vector, and to load a spilled register
// waits for every load and store in flight.  Without spills, 16384 x 1024 x 4096, four output tiles per workgroup, us:
// 93.0 -> 91.0, with GELU 104.2 -> 101.7, with the score 95.2 -> 92.1; 12288 x 768 x 3072 with GELU 64.3 -> 61.6.
__device__ __forceinline__ int lane_again() {
  unsigned all = ~0u;
  asm volatile("" : "+s"(all));
  return (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u));
}
template <int FM, int FN>
__device__ __forceinline__ void acc_ready(v4i (&acc)[FM][FN]) {
  asm volatile("s_nop 15\n\ts_nop 3" ::: "memory");
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) asm volatile("" : "+v"(acc[i][j]));
}

// compile-time loop: f(std::integral_constant<int, I>) for I = FIRST .. LAST - 1
template <int FIRST, int LAST, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (FIRST < LAST) {
    f(std::integral_constant<int, FIRST>{});
    static_for<FIRST + 1, LAST>(f);
  }
}

// The k tile to be requested next: it runs NSTAGE k tiles ahead of the multiplication, across the output tiles of
// the workgroup.  Everything here is wave-uniform.
template <int KB, bool W4>
struct Cursor {
  const char* a;     // first row of its output tile, at its k
  const char* b;     // the workgroup's first W row, at its k
  const char* zero;  // chunks at or beyond `limit` come from here
  int k, limit;      // limit: K; 0 once nothing is left (every further request fetches zeros)
  int tile;

  __device__ __forceinline__ void init(const char* a0, const char* b0, int k_len, int tile_) {
    a = a0;
    b = b0;
    zero = reinterpret_cast<const char*>(g_zero16);
    // once, in scalar registers: left to the compiler it is loaded in front of every request, and the wait for
    // that load (lgkmcnt(0)) drains the LDS reads in flight
    asm volatile("" : "+s"(zero));
    k = 0;
    limit = k_len;
    tile = tile_;
  }
  // The k tile lies inside the row.  An output tile's k loop runs while it does and is followed by one that asks lane by
  // lane (a branch per request in a single loop: 16384 x 4096 x 1024 66.0 us against 62.7, 4096 x 1024 x 1024 11.0 against 10.6)
  __device__ __forceinline__ bool whole() const { return k + KB <= limit; }
  // ... and so does the one after it
  __device__ __forceinline__ bool whole_two(int tile_end) const {
    return k + 2 * KB <= limit || (k + KB == limit && tile + 1 < tile_end);
  }
  // off: the lane's bytes from a (b); kl: its k within the tile
  template <bool WHOLE, bool IS_A>
  __device__ __forceinline__ void fetch(unsigned off, unsigned kl, unsigned lds_byte_off) const {
    const char* base = IS_A ? a : b;
    if (WHOLE) dma16_base(base, off, lds_byte_off);
    else dma16(k + (int)kl < limit ? base + off : zero, lds_byte_off);
  }
  // true: at the first k tile of another output tile, whose rows are the caller's business
  __device__ __forceinline__ bool advance(int tile_end) {
    k += KB;
    a += KB;
    b += W4 ? KB / 2 : KB;
    if (k < limit) return false;
    if (limit == 0 || tile + 1 >= tile_end) {
      limit = 0;
      return false;
    }
    ++tile;
    k = 0;
    return true;
  }
};

// What one wave fetches per stage.  Wave-load t of a wave covers tile rows first + t * STEP ..., and
// because STEP is a multiple of the swizzle period every one of them has the lane fetch the same
// logical chunk.  The offsets do not change with k.
template <class C, bool W4>
struct DmaPlan {
  static constexpr int NA = C::NLA / C::NW, NB = C::NLB / C::NW;
  static constexpr int BRPI = W4 ? C::PRPI : C::RPI;
  static constexpr int STEP_A = C::RPI * C::NW, STEP_B = BRPI * C::NW;
  static_assert(((STEP_A >> C::SH) % C::CPR) == 0, "A swizzle must repeat from one wave-load to the next");
  static_assert(W4 ? ((STEP_B >> C::PSH) % C::PCPR) == 0 : ((STEP_B >> C::SH) % C::CPR) == 0,
                "W swizzle must repeat from one wave-load to the next");
  unsigned off_a[NA], off_b[NB];  // bytes from the tile's first row at k = 0
  unsigned ka, kb;                // k of the lane's chunk within the tile
  unsigned lds_off;               // of the wave's first wave-load within a stage's operand

  // last: last valid row, counted from the tile's first; rows past it re-read it and are never stored
  __device__ __forceinline__ void rows_a(int wave, int lane, unsigned K, unsigned last) {
#pragma unroll
    for (int t = 0; t < NA; ++t) {
      const unsigned row = (unsigned)(C::RPI * wave + lane / C::CPR + t * STEP_A);
      off_a[t] = (row < last ? row : last) * K + ka;
    }
  }
  __device__ __forceinline__ void init(int wave, int lane, unsigned K, unsigned last_b) {
    lds_off = (unsigned)wave * 1024u;
    const int row = C::RPI * wave + lane / C::CPR;
    ka = (unsigned)(((lane % C::CPR) ^ ((row >> C::SH) & (C::CPR - 1))) * 16);
    const int rb = BRPI * wave + (W4 ? lane / C::PCPR : lane / C::CPR);
    kb = W4 ? (unsigned)(((lane % C::PCPR) ^ ((rb >> C::PSH) & (C::PCPR - 1))) * 32) : ka;  // a packed chunk is 32 values
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const unsigned r = (unsigned)(rb + t * STEP_B);
      off_b[t] = (r < last_b ? r : last_b) * (W4 ? K >> 1 : K) + (W4 ? kb >> 1 : kb);
    }
  }
  // request R of the cursor's k tile, numbered 0 .. NA + NB - 1 (A first), into the stage at LDS byte `stage`
  template <int R, bool WHOLE>
  __device__ __forceinline__ void request(const Cursor<C::DBK, W4>& c, unsigned stage) const {
    if constexpr (R < NA) c.template fetch<WHOLE, true>(off_a[R], ka, stage + lds_off + (unsigned)(R * C::NW) * 1024u);
    else c.template fetch<WHOLE, false>(off_b[R - NA], kb, stage + (unsigned)C::A_STAGE + lds_off + (unsigned)((R - NA) * C::NW) * 1024u);
  }
};

// LDS offsets (within a stage) of the first operand fragments of a lane, for k substep 0.  With
// the XOR swizzle the offset for substep s is this value with a compile-time constant XORed into its
// chunk bits, and rows 16 i further down add a multiple of the row pitch, which never reaches those bits.
//
// Which 16 k-values a lane's operand holds in substep s (64 k) is free as long as both operands agree (a
// dot product does not care about the order of its terms).  int8 weights: the natural order, lane
// quarter q of substep s holds k = 64 s + 16 q ..., i.e. 16-byte chunk 4 s + q of both rows.
// Packed int4 weights: a 16-byte LDS chunk holds 32 k-values, and only whole chunks can be read without
// bank conflicts (64-bit reads of half chunks leave half of the banks idle and collide two-fold on
// the rest).  So a lane reads chunk 4 p + j of the W row ONCE per pair p of substeps and multiplies
// its low 8 bytes (k = 128 p + 32 j ...) in substep 2 p, its high 8 bytes (k = 128 p + 32 j + 16 ...) in
// substep 2 p + 1; the A operand follows: chunk 8 p + 2 j + h in substep 2 p + h.  Quarter q takes j = 0, 3, 1, 2:
// the two quarters of either half wave then differ in bits 1 and 2 of their A chunk, which keeps the A reads free of
// bank conflicts whichever 16 of the half wave's lanes are served together.
template <class C, bool W4>
struct FragBase {
  unsigned a, b;
  __device__ __forceinline__ void init(int wm, int wn, int lane) {
    const int r = lane & 15, q = lane >> 4;
    const int j = q == 0 ? 0 : q == 1 ? 3 : q - 1;  // 0 3 1 2
    const int ra = wm * C::TM + r;
    const int ga = W4 ? j << 1 : q;
    a = (unsigned)(ra * C::DBK + ((ga ^ ((ra >> C::SH) & (C::CPR - 1))) << 4));
    const int rb = wn * C::TN + r;
    if (!W4) b = (unsigned)(C::A_STAGE + rb * C::DBK + ((q ^ ((rb >> C::SH) & (C::CPR - 1))) << 4));
    else b = (unsigned)(C::A_STAGE + rb * (C::DBK / 2) + ((j ^ ((rb >> C::PSH) & (C::PCPR - 1))) << 4));
  }
};

// Half H of 32 packed nibbles (see FragBase) as a matrix operand
template <int H>
__device__ __forceinline__ v4i expand_half(const v4i& r) {
  unsigned b0, b1, b2, b3;
  expand8((unsigned)(H ? r.z : r.x), b0, b1);
  expand8((unsigned)(H ? r.w : r.y), b2, b3);
  v4i b = v4i{(int)b0, (int)b1, (int)b2, (int)b3};
  asm volatile("s_nop 1" : "+v"(b));  // see mma
  return b;
}

// A group of four n that lies inside the row travels in one access whatever its alignment.  (A type that came
// through a template argument would have lost its own alignment.)
template <bool VEC>
struct Four {  // N % 4 == 0 and 16-byte aligned outputs
  typedef v4f F;
  typedef v4i I;
  typedef unsigned C;
};
template <>
struct Four<false> {
  typedef f4_any F;
  typedef v4i_any I;
  typedef u32_any C;
};

// What a workgroup does with the accumulators of one output tile (see EpiArgs for EPI).  16x16 accumulator tile
// (i, j): lane l holds m = l % 16 and the four consecutive n = 4 (l / 16) + 0..3: a store instruction writes 64
// bytes of each of 16 rows.  (In 32x32 tiles it is 32 bytes of 32 rows: 67 MB stored by one workgroup per CU 14.5 us
// against 11.5, 16.8 MB in 128 x 128 tiles 6.2 against 4.8, whole rows no better.)
// scales: the tile's per-channel W scales in LDS.  sse, amax: the lane's running sums.
// Rows of N % 4 != 0 values, stored one by one before: 6846 x 1152 x 3139 121 -> 49 us, 2999 x 1152 x 1021 20.8 -> 9.7.
template <class C, bool W4, bool VEC, int EPI, int ACT_KIND>
__device__ __forceinline__ void epilogue_act(const v4i (&acc)[C::FM][C::FN], int64_t cur_m0, int64_t cur_n0, int wm, int wn, int lane,
                                         const char* scales, int64_t M, int64_t N, float sa, bool want_y, float q_inv, float q_max,
                                         float* __restrict__ Y, int32_t* __restrict__ ACC, const EpiArgs& epi, float& sse,
                                         float& amax) {
  constexpr bool SCORE = EPI == 1, ACT = EPI >= 2, AMAX = EPI == 2, QOUT = EPI == 3;
  int8_t* __restrict__ CODES = epi.codes;
  const float* __restrict__ YREF = epi.yref;
  using F4 = typename Four<VEC>::F;
  using I4 = typename Four<VEC>::I;
  using C4 = typename Four<VEC>::C;
  static_assert(alignof(F4) == (VEC ? 16 : 4) && alignof(I4) == (VEC ? 16 : 4) && alignof(C4) == (VEC ? 4 : 1),
                "no access promises more than the address has");
  const int nq = wn * C::TN + (lane >> 4) * 4;  // the lane's first n within the tile
  // Score: the loads of four accumulator tiles are in flight together, two rows of them where a row has two (past the edge:
  // others of the matrix).  us, two in flight | four, operands from memory, M x K x N: 6301 x 128 x 60
  // 6.8 | 6.3, 5272 x 288 x 72 7.5 | 7.1, 15489 x 160 x 192 10.6 | 10.1, 4737 x 724 x 51 10.3 | 9.7.  (In the aligned
  // 64 tile the compiler moves two of them behind the first row's arithmetic; held in front of it all are 1-2 % slower.)
  constexpr int G = C::FN % 4 == 0 ? 4 : 2, GI = 4 / G;
  static_assert(C::FN % 2 == 0 && C::FM % GI == 0, "groups of four accumulator tiles");
#pragma unroll
  for (int i0 = 0; i0 < C::FM; i0 += GI) {
#pragma unroll
    for (int j0 = 0; j0 < C::FN; j0 += G) {
      v4f yref[GI][G];
      if (SCORE && (VEC || N >= 4)) {
#pragma unroll
        for (int h = 0; h < GI; ++h) {
          const int64_t m = cur_m0 + wm * C::TM + (i0 + h) * 16 + (lane & 15);
          const float* row = YREF + (m < M ? m : cur_m0) * N;
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const int64_t n = cur_n0 + nq + (j0 + g) * 16;
            yref[h][g] = *reinterpret_cast<const F4*>(row + (n + 4 <= N ? n : 0));
          }
        }
      }
#pragma unroll
      for (int h = 0; h < GI; ++h) {
        const int i = i0 + h;
        const int64_t m = cur_m0 + wm * C::TM + i * 16 + (lane & 15);
        if (m >= M) continue;
        float part = 0.0f;  // the row's squares of the group, summed before they join the lane's running sum: short chains
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const int j = j0 + g;
          const int64_t n = cur_n0 + nq + j * 16;
          if (n >= N) continue;
          int a[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            a[e] = acc[i][j][e];
            if (W4) a[e] >>= 4;  // exact: every product carried the factor 16
          }
          const float4 sw = *reinterpret_cast<const float4*>(scales + (nq + j * 16) * 4);
          if (VEC || n + 4 <= N) {  // VEC: N % 4 == 0 and 16-byte aligned outputs
            if (EPI == 0 && ACC) *reinterpret_cast<I4*>(ACC + m * N + n) = v4i{a[0], a[1], a[2], a[3]};
            if (want_y) {
              float4 y = make_float4(((float)a[0] * sa) * sw.x, ((float)a[1] * sa) * sw.y,
                                     ((float)a[2] * sa) * sw.z, ((float)a[3] * sa) * sw.w);
              if (ACT) {
                y = apply_act4(y, ACT_KIND);
                if (AMAX) amax = fmaxf(fmaxf(amax, fmaxf(fabsf(y.x), fabsf(y.y))), fmaxf(fabsf(y.z), fabsf(y.w)));
              }
              if (!QOUT && Y) *reinterpret_cast<F4*>(Y + m * N + n) = v4f{y.x, y.y, y.z, y.w};
              if (QOUT && CODES) {  // four codes, lowest n in the lowest byte
                const unsigned c0 = (unsigned)(int)code_f(y.x, q_inv, q_max) & 0xFFu;
                const unsigned c1 = (unsigned)(int)code_f(y.y, q_inv, q_max) & 0xFFu;
                const unsigned c2 = (unsigned)(int)code_f(y.z, q_inv, q_max) & 0xFFu;
                const unsigned c3 = (unsigned)(int)code_f(y.w, q_inv, q_max);
                *reinterpret_cast<C4*>(CODES + m * N + n) = c0 | (c1 << 8) | (c2 << 16) | (c3 << 24);
              }
              if (SCORE) {
                const v4f r = yref[h][g];
                float d = y.x - r.x;
                part = __builtin_fmaf(d, d, part);
                d = y.y - r.y;
                part = __builtin_fmaf(d, d, part);
                d = y.z - r.z;
                part = __builtin_fmaf(d, d, part);
                d = y.w - r.w;
                part = __builtin_fmaf(d, d, part);
              }
            }
          } else {  // the last group of a row that it does not fill
            const float s4[4] = {sw.x, sw.y, sw.z, sw.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              if (n + e >= N) break;
              if (EPI == 0 && ACC) ACC[m * N + n + e] = a[e];
              if (want_y) {
                float y = ((float)a[e] * sa) * s4[e];
                if (ACT) {
                  y = apply_act(y, ACT_KIND);
                  if (AMAX) amax = fmaxf(amax, fabsf(y));
                }
                if (!QOUT && Y) Y[m * N + n + e] = y;
                if (QOUT && CODES) CODES[m * N + n + e] = (int8_t)(int)code_f(y, q_inv, q_max);
                if (SCORE && YREF) {
                  const float d = y - YREF[m * N + n + e];
                  part = __builtin_fmaf(d, d, part);
                }
              }
            }
          }
        }
        if (SCORE) sse += part;
      }
    }
  }
}

// The kind of activation is chosen once per output tile: with a uniform branch per four values 4096 x 1024 x 1024 with
// ReLU spends 2.3 us between its last matrix step and its last store, against 1.15 without an activation.
template <class C, bool W4, bool VEC, int EPI>
__device__ __forceinline__ void epilogue(const v4i (&acc)[C::FM][C::FN], int64_t cur_m0, int64_t cur_n0, int wm, int wn, int lane,
                                         const char* scales, int64_t M, int64_t N, float sa, bool want_y, float q_inv, float q_max,
                                         float* __restrict__ Y, int32_t* __restrict__ ACC, const EpiArgs& epi, float& sse,
                                         float& amax) {
#define MPQ_EPI(K_)                                                                                                     \
  epilogue_act<C, W4, VEC, EPI, K_>(acc, cur_m0, cur_n0, wm, wn, lane, scales, M, N, sa, want_y, q_inv, q_max, Y, ACC, epi, sse, amax)
  if (EPI >= 2 && epi.act == 2) MPQ_EPI(2);
  else if (EPI >= 2 && epi.act == 1) MPQ_EPI(1);
  else MPQ_EPI(0);
#undef MPQ_EPI
}

// The workgroup's share of the score or of the running maximum, once its last output tile is done.  index: its number.
template <class C, int EPI>
__device__ __forceinline__ void finish_sums(char* lds, int wave, float sse, float amax, const EpiArgs& epi,
                                            int64_t index) {
  float* sm = reinterpret_cast<float*>(lds + C::SUMS_OFF);
  const int lane = lane_again();
  if (EPI == 1 && epi.part) {  // one partial per workgroup, combined in a fixed order
    const float w = wave_sum(sse);
    if (lane == 0) sm[wave] = w;
    lds_done();
    meet();
    if (wave == 0 && lane == 0) {
      double t = 0.0;
      for (int i = 0; i < C::NW; ++i) t += (double)sm[i];
      epi.part[index] = t;
    }
  }
  if (EPI == 2 && epi.amax) {  // one atomic per workgroup
    const float w = wave_max(amax);
    if (lane == 0) sm[wave] = w;
    lds_done();
    meet();
    if (wave == 0 && lane == 0) {
      float t = 0.0f;
      for (int i = 0; i < C::NW; ++i) t = fmaxf(t, sm[i]);
      if (epi.amax_part) epi.amax_part[index] = t;
      else atomicMax(epi.amax, abs_key(t));
    }
  }
}

// A workgroup works off `chunk` output tiles that follow each other along M (same columns, so
// the W tile stays hot and, at any moment, the workgroups in flight still write all column blocks
// of Y: tiles that follow each other along N made the whole grid store into the same quarter of
// every Y row at the same time, which the memory channels punish).  Workgroup ids run with N
// fastest; `remap` regroups them so that the workgroups an XCD receives (ids congruent mod 8)
// cover a contiguous id range and share its L2.
// The k loop never drains between the tiles of a chunk: the requests issued during the last k
// tiles of one output tile already fetch the first k tiles of the next one.  Chunks stay short so that the
// hardware dispatcher, not a fixed assignment, balances the load when other kernels hold some of the CUs.
// MINW: waves the register allocation must leave room for on one SIMD.
// EPI: 0 plain, 1 score, 2 activation and absmax of the output, 3 activation and int8 codes of the
// output (see EpiArgs); variants of their own because the largest tile has no registers to spare
// for them in the plain kernel.
template <int BM, int BN, int WM, int WN, int NSTAGE, bool W4, bool VEC, int KB, int MINW, int EPI>
__global__ __launch_bounds__(WM * WN * 64, MINW) void qgemm_dma(const int8_t* __restrict__ A,
                                                          const void* __restrict__ Wv, int64_t M,
                                                          int64_t N, int64_t K,
                                                          const float* __restrict__ a_scale,
                                                          const float* __restrict__ w_scale,
                                                          int w_per_row, float* __restrict__ Y,
                                                          int32_t* __restrict__ ACC, EpiArgs epi,
                                                          int tiles_n, int tiles_m, int chunk,
                                                          int remap, int k_per_split) {
  constexpr bool QOUT = EPI == 3;
  using C = DmaCfg<BM, BN, WM, WN, NSTAGE, W4, KB>;
  using P = DmaPlan<C, W4>;
  constexpr int NSUB = KB / 64;
  static_assert(NSUB % 2 == 0, "operand registers alternate from one k substep to the next");
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wm = wave / WN, wn = wave % WN;
  const unsigned lds0 = (unsigned)(uintptr_t)MPQ_LPTR(lds);  // LDS byte address of the buffer
  const int G = (int)gridDim.x;
  int wg = (int)blockIdx.x;
  if (remap) wg = (wg & 7) * (G >> 3) + (wg >> 3);  // G % 8 == 0
  // Split along k (gridDim.y > 1): workgroup row y takes k in [y * k_per_split, ...) and leaves its
  // raw accumulators in plane y of ACC; the caller adds the planes up (integers: exact in any order).
  const int k_begin = (int)blockIdx.y * k_per_split;  // a multiple of the k tile; 0 without a split
  const int k_len = ((int)K - k_begin < k_per_split) ? (int)K - k_begin : k_per_split;
  if (gridDim.y > 1) {
    A += k_begin;
    Wv = reinterpret_cast<const char*>(Wv) + (W4 ? k_begin >> 1 : k_begin);
    ACC += (int64_t)blockIdx.y * M * N;
  }
  const int KT = (k_len + KB - 1) / KB;
  int tile = (wg / tiles_n) * chunk;  // row of tiles; < tiles_m: the grid is ceil(tiles_m / chunk) * tiles_n
  const int tile_end = tile + chunk < tiles_m ? tile + chunk : tiles_m;
  const int64_t n0 = (int64_t)(wg % tiles_n) * BN;
  const bool want_y = EPI != 0 || Y != nullptr;

  P plan;
  plan.init(wave, lane, (unsigned)K, (unsigned)(N - 1 - n0 < BN ? N - 1 - n0 : BN));
  const char* const b_first = reinterpret_cast<const char*>(Wv) + n0 * (W4 ? K >> 1 : K);
  Cursor<KB, W4> cursor;
  cursor.init(nullptr, b_first, k_len, tile);
  // The lane's offsets are the same in every output tile but one that reaches past M, which is the workgroup's last.
  // (Formed for each tile they were known before the k loop and spilled over it by the 256 tile, and to load a spilled
  // register waits for all stores in flight: with the epilogue's addresses, below, 16384 x 1024 x 4096 95.2 -> 91.3 us.)
  auto start_rows = [&](bool first) {
    const int64_t m = (int64_t)cursor.tile * BM;
    cursor.a = reinterpret_cast<const char*>(A) + m * K;
    cursor.b = b_first;
    if (first || m + BM > M) plan.rows_a(wave, first ? lane : lane_again(), (unsigned)K, (unsigned)(M - 1 - m < BM ? M - 1 - m : BM));
  };
  start_rows(true);
  if (want_y && w_per_row) request_scales<VEC>(w_scale, n0, N, BN, lane, lds0 + C::SCALE_OFF);
#pragma unroll
  for (int p = 0; p < NSTAGE; ++p) {
    if (cursor.whole()) static_for<0, C::LPW>([&](auto r_) { plan.template request<decltype(r_)::value, true>(cursor, lds0 + p * C::STAGE); });
    else static_for<0, C::LPW>([&](auto r_) { plan.template request<decltype(r_)::value, false>(cursor, lds0 + p * C::STAGE); });
    if (cursor.advance(tile_end)) start_rows(false);
  }
  // The scalars of the epilogue are loaded here, behind the requests, once, into scalar registers.  (Loaded in the
  // epilogue they may come as vector loads whose arrival the compiler waits for at every store, vmcnt(0), as it
  // cannot tell on which path they were used first, and stores count in vmcnt as well: each 16-byte store of a
  // wave then waits for the one before it to be acknowledged.)
  const float sa = want_y ? load_scalar(a_scale) : 0.0f, sw0 = want_y && !w_per_row ? load_scalar(w_scale) : 0.0f;
  float q_inv = 0.0f, q_max = 0.0f;
  if (QOUT) {
    float q_scale;
    bit_constants(load_scalar(epi.q_absmax), epi.q_bits, q_scale, q_inv);
    q_max = (float)((1 << (epi.q_bits - 1)) - 1);
  }
  if (want_y && !w_per_row) {
    float* sc = reinterpret_cast<float*>(lds + C::SCALE_OFF);
    for (int i = threadIdx.x; i < 256; i += C::NT) sc[i] = sw0;
  }

  // Operand registers of two k substeps (64 k each): one set is multiplied while the other is read from LDS.
  // Packed weights are read once per pair of substeps and expanded, both halves, during the first of them.
  v4i fa[2][C::FM], fb[2][C::FN], raw[W4 ? C::FN : 1];
  FragBase<C, W4> fr;
  fr.init(wm, wn, lane);
  auto lds_at = [&](unsigned off) { return *reinterpret_cast<const v4i*>(lds + off); };
  // reads of substep S of the stage at `stage`, numbered so that the first matrix step's operands come first
  auto read = [&](auto s_, auto n_, unsigned stage) {
    constexpr int S = decltype(s_)::value, n = decltype(n_)::value;
    // chunk bits: 4 S + q (int8 weights) or 8 (S / 2) + 2 j + S % 2 (packed weights); q and j are in fr
    constexpr unsigned xa = W4 ? (unsigned)(((S >> 1) << 7) | ((S & 1) << 4)) : (unsigned)(S << 6);
    constexpr unsigned xb = W4 ? (unsigned)((S >> 1) << 6) : (unsigned)(S << 6);
    if constexpr (n < C::FM) fa[S & 1][n] = lds_at(((fr.a + stage) ^ xa) + (unsigned)(n * 16 * C::DBK));
    else if constexpr (W4) raw[n - C::FM] = lds_at(((fr.b + stage) ^ xb) + (unsigned)((n - C::FM) * 16 * C::B_ROW));
    else fb[S & 1][n - C::FM] = lds_at(((fr.b + stage) ^ xb) + (unsigned)((n - C::FM) * 16 * C::B_ROW));
  };

  wait_vmcnt<(NSTAGE - 1) * C::LPW>();  // this wave's share of k tile 0 has landed
  float sse = 0.0f;   // this lane's share of sum (Y - YREF)^2 over the chunk
  float amax = 0.0f;  // this lane's largest |Y| after the activation
  unsigned cur = 0;   // stage of the k tile being multiplied
  int landed = 0;     // k tiles of this output tile known to be in LDS already

  while (true) {
    // Everyone's share of the first k tile is there.  (Its operands are read here and not carried over from the loop
    // before: they would hold registers that the epilogue needs.)
    lds_done();
    meet();
    static_for<0, C::FM + C::FN>([&](auto n_) { read(std::integral_constant<int, 0>{}, n_, cur); });
    v4i acc[C::FM][C::FN];
    zero_acc(acc);
    auto step = [&](auto whole_, int t) {
      unsigned nxt = cur + C::STAGE;
      nxt = nxt == NSTAGE * C::STAGE ? 0u : nxt;
      static_for<0, NSUB>([&](auto sub_) {
        constexpr int S = decltype(sub_)::value;
        constexpr bool LAST = S == NSUB - 1;
        constexpr int S1 = LAST ? 0 : S + 1;  // whose operands are read meanwhile, two per matrix step
        constexpr int NR = C::FM + (W4 && (S1 & 1) ? 0 : C::FN), NM = C::FM * C::FN, NQ = LAST ? C::LPW : 0;
        // The stage has been read for the last time and the next k tile has landed: its first operands are read and
        // the stage is filled again while this substep, whose operands are in registers, is multiplied.
        if constexpr (LAST) {
          lds_done();
          if (t + 1 >= landed) wait_vmcnt<(NSTAGE - 2) * C::LPW>();
          meet();
        }
        if constexpr (W4 && (S & 1) == 0) fb[0][0] = expand_half<0>(raw[0]);
        static_for<0, NM>([&](auto m_) {
          constexpr int m = decltype(m_)::value, j = m / C::FM, i = m % C::FM;
          // W fragment as the row operand: the lane then holds 4 consecutive n, which the epilogue stores as one
          // 16-byte piece of a Y row
          mma(acc[i][j], fb[S & 1][j], fa[S & 1][i]);
          __builtin_amdgcn_sched_barrier(0);
          static_for<2 * m < NR ? 2 * m : NR, 2 * m + 2 < NR ? 2 * m + 2 : NR>(
              [&](auto n_) { read(std::integral_constant<int, S1>{}, n_, LAST ? nxt : cur); });
          static_for<m * NQ / NM, (m + 1) * NQ / NM>([&](auto r_) { plan.template request<decltype(r_)::value, decltype(whole_)::value>(cursor, lds0 + cur); });
          if constexpr (W4 && (S & 1) == 0 && i == 0) fb[1][j] = expand_half<1>(raw[j]);
          if constexpr (W4 && (S & 1) == 0 && i == C::FM - 1 && j + 1 < C::FN) fb[0][j + 1] = expand_half<0>(raw[j + 1]);
          __builtin_amdgcn_sched_barrier(0);
        });
      });
      if (cursor.advance(tile_end)) start_rows(false);
      cur = nxt;
    };
    int t = 0;
    for (; t < KT && cursor.whole(); ++t) step(std::true_type{}, t);
    for (; t < KT; ++t) step(std::false_type{}, t);
    // The next output tile's first NSTAGE k tiles land here, ahead of the stores: no wait of its first barriers
    // then has to wait for a store (both count in vmcnt).  Behind the last output tile only zeros are on their way, and
    // its stores do not wait for them (us, before | now, M x K x N: 11799 x 160 x 72 4.62 | 4.43, with the score and operands
    // from memory 4928 x 64 x 512 9.35 | 8.52, 3574 x 704 x 320 10.6 | 10.1; the 256 tile, whose last wait is a smaller part, is
    // no faster and waits).
    const bool last = tile + 1 >= tile_end;  // block-uniform
    if (!last) wait_vmcnt<0>();
    landed = NSTAGE;
    acc_ready(acc);
    epilogue<C, W4, VEC, EPI>(acc, (int64_t)tile * BM, n0, wm, wn, lane_again(), lds + C::SCALE_OFF, M, N, sa, want_y, q_inv, q_max,
                              Y, ACC, epi, sse, amax);
    if (last) break;
    ++tile;
  }
  finish_sums<C, EPI>(lds, wave, sse, amax, epi, blockIdx.x);
  wait_vmcnt<0>();  // the zeros, before the LDS is given back
}

// Dynamic LDS above 64 KiB has to be allowed once per kernel and device (hipFuncSetAttribute, not a
// stream operation).  `done` is one flag word per device, a bit per kernel variant of the caller's
// instantiation; setting the attribute twice is harmless, so a relaxed flag is all the
// synchronisation two host threads racing through here need.
constexpr int kMaxDevices = 64;
inline int allow_lds(const void* kern, int bytes, std::atomic<unsigned>* done, int which) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) dev = 0;
  if (done[dev].load(std::memory_order_relaxed) & (1u << which)) return MPQ_OK;
  hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) { set_last_hip_error((int)e); return MPQ_ERR_HIP; }
  done[dev].fetch_or(1u << which, std::memory_order_relaxed);
  return MPQ_OK;
}

// How a call is launched with a tile size: kernel variant (EPI * 2 + VEC), grid and chunk length.
struct LaunchShape {
  int which = 0;
  int64_t tm = 0, tn = 0, grid = 0;
  int chunk = 1, remap = 0;
};
inline int launch_shape(int bm, int bn, int lds_bytes, int64_t M, int64_t N, const float* w_scale, int per_row, const float* y_out,
                        const int32_t* acc_out, const EpiArgs& epi, int split, LaunchShape& s) {
  // float4 / int4 stores need every 4-group of n inside the row and 16-byte aligned
  const bool vec = (N & 3) == 0 && (!y_out || aligned16(y_out)) && (!acc_out || aligned16(acc_out)) &&
                   (!((y_out || epi.yref || epi.amax || epi.codes) && per_row) || aligned16(w_scale)) &&
                   (!epi.yref || aligned16(epi.yref)) && (!epi.codes || (reinterpret_cast<uintptr_t>(epi.codes) & 3u) == 0);
  const int mode = epi.yref ? 1 : epi.codes ? 3 : (epi.act || epi.amax) ? 2 : 0;
  s.which = mode * 2 + (vec ? 1 : 0);
  s.tm = (M + bm - 1) / bm;
  s.tn = (N + bn - 1) / bn;
  if (s.tm * s.tn > 0x7FFFFFFF || s.tn > 0x7FFFFFFF) return MPQ_ERR_SHAPE;
  s.chunk = chunk_tiles(s.tm, s.tn, split, lds_bytes, kNumCU);
  s.grid = (s.tm + s.chunk - 1) / s.chunk * s.tn;
  s.remap = (s.grid % 8 == 0 && s.grid >= 16) ? 1 : 0;
  return MPQ_OK;
}

// prepare_only: configure every kernel variant of this instantiation and launch nothing (mpq_init).
// split > 1: workgroup rows y = 0 .. split - 1 each take k_per_split of k (a multiple of the k tile)
// and write raw accumulators to plane y of acc_out (plain epilogue only).
template <int BM, int BN, int WM, int WN, int NSTAGE, bool W4, int KB = 128, int MINW = 1>
static int launch_dma(const int8_t* a_q, const void* w_q, int64_t M, int64_t N, int64_t K,
                      const float* a_scale, const float* w_scale, int per_row, float* y_out,
                      int32_t* acc_out, hipStream_t st, EpiArgs epi = kNoEpi,
                      int64_t* n_partials = nullptr, int split = 1, int k_per_split = 0,
                      bool prepare_only = false) {
  using C = DmaCfg<BM, BN, WM, WN, NSTAGE, W4, KB>;
  using Kern = void (*)(const int8_t*, const void*, int64_t, int64_t, int64_t, const float*, const float*, int,
                        float*, int32_t*, EpiArgs, int, int, int, int, int);
  static const Kern kerns[8] = {
      qgemm_dma<BM, BN, WM, WN, NSTAGE, W4, false, KB, MINW, 0>, qgemm_dma<BM, BN, WM, WN, NSTAGE, W4, true, KB, MINW, 0>,
      qgemm_dma<BM, BN, WM, WN, NSTAGE, W4, false, KB, MINW, 1>, qgemm_dma<BM, BN, WM, WN, NSTAGE, W4, true, KB, MINW, 1>,
      qgemm_dma<BM, BN, WM, WN, NSTAGE, W4, false, KB, MINW, 2>, qgemm_dma<BM, BN, WM, WN, NSTAGE, W4, true, KB, MINW, 2>,
      qgemm_dma<BM, BN, WM, WN, NSTAGE, W4, false, KB, MINW, 3>, qgemm_dma<BM, BN, WM, WN, NSTAGE, W4, true, KB, MINW, 3>};
  static std::atomic<unsigned> done[kMaxDevices];
  if (prepare_only) {
    for (int w = 0; w < 8; ++w) {
      const int rc = allow_lds(reinterpret_cast<const void*>(kerns[w]), C::LDS_BYTES, done, w);
      if (rc != MPQ_OK) return rc;
    }
    return MPQ_OK;
  }
  if (split <= 1) { split = 1; k_per_split = (int)K; }
  LaunchShape s;
  int rc = launch_shape(BM, BN, C::LDS_BYTES, M, N, w_scale, per_row, y_out, acc_out, epi, split, s);
  if (rc == MPQ_OK) rc = allow_lds(reinterpret_cast<const void*>(kerns[s.which]), C::LDS_BYTES, done, s.which);
  if (rc != MPQ_OK) return rc;
  kerns[s.which]<<<dim3((unsigned)s.grid, (unsigned)split), C::NT, C::LDS_BYTES, st>>>(
      a_q, w_q, M, N, K, a_scale, w_scale, per_row, y_out, acc_out, epi, (int)s.tn, (int)s.tm, s.chunk, s.remap, k_per_split);
  if (n_partials) *n_partials = s.grid;
  return launch_status();
}

// What a translation unit of one tile size exports: validation is the caller's business.
struct DmaArgs {
  const int8_t* a_q;
  const void* w_q;
  int64_t M, N, K;
  const float* a_scale;
  const float* w_scale;
  int per_row;
  float* y_out;
  int32_t* acc_out;
  hipStream_t st;
  EpiArgs epi;
  int64_t* n_partials;
  int split;         // > 1: split along k, raw accumulators to `split` planes of acc_out
  int k_per_split;
  bool prepare_only;  // configure the kernels of this tile size, launch nothing
};
int launch_dma_256(bool w4, const DmaArgs& a);
int launch_dma_192(bool w4, int stages, const DmaArgs& a);
int launch_dma_128(bool w4, int stages, const DmaArgs& a);
int launch_dma_64(bool w4, int stages, int kb, const DmaArgs& a);

// Layers with few output tiles (qgemm_skinny.hip): how many waves split k, 0 where the layer is better
// off with the tiled kernels.
int skinny_waves(int64_t M, int64_t N, int64_t K, bool amax);
int launch_skinny(int waves, bool w4, const DmaArgs& d);

}  // namespace mpq
