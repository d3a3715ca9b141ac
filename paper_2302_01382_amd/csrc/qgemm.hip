// qgemm.hip -- one quantized linear layer, the dense core of the evaluation step in the paper's
// Alg. 1 / Alg. 2: acc[m][n] = sum_k A_q[m][k] * W_q[n][k] in int32 on the int8 matrix cores,
// then Y = (float(acc) * s_A) * s_W[n].
//
// Both operands are K-contiguous, which is exactly what the int8 matrix instructions want: a lane of
// either operand holds 16 consecutive k-bytes of a tile row.
//
// Three kernels: the fast path (qgemm_dma.hpp and qgemm_quad.hpp; 16-byte aligned operands, K a multiple of 16, or 32
// for packed int4) feeds a multi-stage LDS pipeline with direct global->LDS loads; qgemm_any right
// below stages tiles through registers and handles any K and alignment; qgemm_skinny.hip takes layers of few
// output tiles.  Same arithmetic, same results.
//
// Packed int4 weights are expanded on their way to the matrix core: a nibble n becomes the byte
// n << 4 (= 16 n as int8, sign included), so the accumulator holds 16 * acc exactly and is shifted
// back by 4.
#include "qgemm_dma.hpp"

namespace mpq {

__global__ void fill_u32_k(unsigned* p, unsigned v) { p[0] = v; }

// =====================================================================================================
// Any K, any alignment: tiles staged through registers.
//
// Rows of a tensor with K % 16 != 0 start at any byte, so a tile cannot travel by global->LDS loads of
// 16 aligned bytes.  A thread fetches its chunks of 16 bytes into registers (AnyStage), up to three k tiles of 128
// ahead, and writes them to a double-buffered LDS tile; one barrier per k tile.  The loads of k tiles behind the last one
// are issued as well, at the row's last bytes: nothing outside the row's dwords is ever read.
//
// What bounds it: a k tile's chain of loads, stores, barrier, reads and matrix steps, which the other workgroups of the CU
// hide in part, and the output (stored value by value it was as long as eight k tiles).  us, before the chunks were loaded
// as dwords, the output stored in 16 bytes and the 128 tile given eight waves -> now (M x K x N): 2999 x 1155 x 1021
// 19.9 -> 14.7, 16384 x 1001 x 1000 59.5 -> 55, 512 x 1001 x 512 8.7 -> 6.9, 4000 x 2002 x 1500 42 -> 34, 6272 x 2302 x 256
// packed 18.7 -> 16.5, 3000 x 1156 x 1000 16.3 -> 12.6; an aligned 2999 x 1152 x 1021 takes 9.7 on the fast path.  Chunks
// written between the matrix steps instead of in front of the barrier: 15.8 -> 17.0.
// The 64 tile keeps within 128 registers, four workgroups per CU: with 136 (int8 weights, rows at any byte: an address and a
// shift per chunk) there were three, and 2000 x 250 x 2000, 1024 tiles, took two rounds: 10.9 us against 9.2, 4096 x 33 x 1000
// 8.9 against 7.3, 1900 x 130 x 2048 10.7 against 8.9.
// =====================================================================================================
constexpr int kAnyBK = 128;       // k values per tile

// byte offset of 16-byte chunk `ch` (0..7) of tile row `row` in a [rows][128 B] LDS tile; the XOR makes
// the 16 lanes served per clock (one chunk column of 16 rows) distinct modulo 256 B (64 banks)
__device__ __forceinline__ int lds_off(int row, int ch) { return row * kAnyBK + ((ch ^ ((row >> 1) & 7)) << 4); }

// One thread's share of an operand tile: CN chunks of 16 bytes, chunk j of tile row row0 + j * STEP.
// CPR: chunks per tile row (8, or 4 of a packed-int4 tile, whose 16 bytes are 32 values).
// A load of 16 bytes per lane runs at 7.5 ns per KiB and CU at any address that is a multiple of 4 and at 17-22 at one
// that is not (measured out of the L2), so the dwords that hold the row's bytes are loaded and shifted into place on
// their way to the LDS.  The dword a chunk lacks at its end comes from the next lane, the last chunk's from the next
// k tile.  Nothing is read but dwords that hold a byte of the row.
// KIND: rows that start at a multiple of 4 (nothing to shift), at any byte, or of less than 16 bytes, which are read byte
// by byte and have a single k tile.
enum RowKind { kRowsDword, kRowsByte, kRowsShort };
template <int NT, int ROWS, int CPR, RowKind KIND>
struct AnyStage {
  static constexpr bool SHORT = KIND == kRowsShort;
  static constexpr int STEP = NT / CPR, CN = ROWS / STEP;
  static_assert(STEP % 4 == 0, "the rows of a thread start at the same byte of their dwords");
  const uint8_t* base;  // the dword that the tile's first row starts in (workgroup-uniform)
  unsigned off[CN];     // of the dwords that the thread's rows start in (SHORT: of the rows), counted from it
  unsigned front;       // bytes of those dwords in front of the row
  int last;             // the last place, counted from them, that 16 bytes of a row's dwords start at
  int kb;               // byte offset of the thread's chunk within a tile row
  int row_bytes;

  __device__ __forceinline__ void init(const void* all, int64_t nrows, int64_t row_bytes_, int64_t r0) {
    row_bytes = (int)row_bytes_;
    kb = ((int)threadIdx.x % CPR) * 16;
    base = reinterpret_cast<const uint8_t*>(all) + r0 * row_bytes_;
    const unsigned skew = KIND == kRowsByte ? (unsigned)reinterpret_cast<uintptr_t>(base) & 3u : 0u;
    base -= skew;
    const unsigned edge_row = (unsigned)(nrows - 1 - r0 < ROWS ? nrows - 1 - r0 : ROWS);
    // rows past the edge re-read the thread's first row, or the last one if that is past it as well; never stored
    const unsigned r = threadIdx.x / CPR, first = r < edge_row ? r : edge_row;
    const unsigned at = first * (unsigned)row_bytes_ + skew;
    front = KIND == kRowsByte ? at & 3u : 0u;
    last = (((int)front + row_bytes + 3) & ~3) - 16;
#pragma unroll
    for (int j = 0; j < CN; ++j) off[j] = at - front + (r + j * STEP <= edge_row ? (unsigned)(j * STEP) * (unsigned)row_bytes_ : 0u);
  }
  // k0: first byte of the tile within the row
  __device__ __forceinline__ void load(v4i (&c)[CN], int k0) const {
    const int k = k0 + kb;
#pragma unroll
    for (int j = 0; j < CN; ++j) {
      if (SHORT) c[j] = load_chunk16(base + off[j], row_bytes, k);
      else c[j] = *reinterpret_cast<const v4i_any*>(base + (off[j] + (unsigned)(k < last ? k : last)));
    }
  }
  // the tile, or with rows at any byte the one after it, reaches the row's end (workgroup-uniform)
  __device__ __forceinline__ bool edge(int k0) const { return k0 + (KIND == kRowsByte ? 2 : 1) * CPR * 16 > row_bytes; }
  // dwords that a load at the row's end was moved back by, zeros behind the end
  __device__ __forceinline__ static v4i moved(v4i c, int back) {
    if (back >= 16) return v4i{0, 0, 0, 0};
    if (back >= 8) c = v4i{c.z, c.w, 0, 0};
    if (back == 4 || back == 12) c = v4i{c.y, c.z, c.w, 0};
    return c;
  }
  // chunk j of the tile at k0, as it goes into the LDS; next: the chunks of the tile after it
  template <bool EDGE>
  __device__ __forceinline__ v4i place(const v4i (&cur)[CN], const v4i (&next)[CN], int j, int k0) const {
    const int k = k0 + kb;
    if constexpr (SHORT) return fix_chunk16(cur[j], row_bytes, k);
    v4i c = cur[j];
    if (EDGE && k > last) c = moved(c, k - last);
    if constexpr (KIND == kRowsDword) return c;
    int follow = next[j].x;
    if (EDGE && k + CPR * 16 > last) follow = moved(next[j], k + CPR * 16 - last).x;
    // the dword behind the chunk: the first of the next lane's; of the last lane of a row the first of the next tile
    const int lane = (int)threadIdx.x % CPR, w = lane == 0 ? follow : c.x;
    int behind;
    if constexpr (CPR == 4) {
      behind = __builtin_amdgcn_update_dpp(0, w, 0x39, 0xF, 0xF, true);  // quad_perm 1 2 3 0
    } else {
      const int up = __builtin_amdgcn_update_dpp(0, w, 0x101, 0xF, 0xF, true);    // row_shl 1: from the lane above
      const int down = __builtin_amdgcn_update_dpp(0, w, 0x117, 0xF, 0xF, true);  // row_shr 7: from seven lanes below
      behind = lane == CPR - 1 ? down : up;
    }
    c = v4i{(int)__builtin_amdgcn_alignbyte((unsigned)c.y, (unsigned)c.x, front),
            (int)__builtin_amdgcn_alignbyte((unsigned)c.z, (unsigned)c.y, front),
            (int)__builtin_amdgcn_alignbyte((unsigned)c.w, (unsigned)c.z, front),
            (int)__builtin_amdgcn_alignbyte((unsigned)behind, (unsigned)c.w, front)};
    if (EDGE) {  // bytes behind the row's end may be the next row's
      auto keep = [](int v, int valid) { return valid >= 4 ? v : valid <= 0 ? 0 : v & (int)((1u << (8 * valid)) - 1u); };
      const int valid = row_bytes - k;
      c = v4i{keep(c.x, valid), keep(c.y, valid - 4), keep(c.z, valid - 8), keep(c.w, valid - 12)};
    }
    return c;
  }
};

template <bool EDGE, class S>
__device__ __forceinline__ void store8(int8_t* lds, const S& st, const v4i (&c)[S::CN], const v4i (&next)[S::CN], int k0) {
  const int row = (int)threadIdx.x >> 3, ch = (int)threadIdx.x & 7;
#pragma unroll
  for (int j = 0; j < S::CN; ++j)
    *reinterpret_cast<v4i*>(lds + lds_off(row + j * S::STEP, ch)) = st.template place<EDGE>(c, next, j, k0);
}

template <bool EDGE, class S>
__device__ __forceinline__ void store4(int8_t* lds, const S& st, const v4i (&c)[S::CN], const v4i (&next)[S::CN], int k0) {
  const int row = (int)threadIdx.x >> 2, quarter = (int)threadIdx.x & 3;
#pragma unroll
  for (int j = 0; j < S::CN; ++j) {
    const v4i v = st.template place<EDGE>(c, next, j, k0);
    unsigned b[8];
    expand8((unsigned)v.x, b[0], b[1]);
    expand8((unsigned)v.y, b[2], b[3]);
    expand8((unsigned)v.z, b[4], b[5]);
    expand8((unsigned)v.w, b[6], b[7]);
    const int r = row + j * S::STEP;
    *reinterpret_cast<v4i*>(lds + lds_off(r, 2 * quarter)) = v4i{(int)b[0], (int)b[1], (int)b[2], (int)b[3]};
    *reinterpret_cast<v4i*>(lds + lds_off(r, 2 * quarter + 1)) = v4i{(int)b[4], (int)b[5], (int)b[6], (int)b[7]};
  }
}

// grid: x = N tiles (fast index, so neighbouring workgroups share the A row panel), y = M tiles.
// TS: side of the output tile: 64 with four waves as 2 x 2, 128 with eight as 2 x 4.  EPI: as qgemm_dma.
template <int TS>
struct AnyCfg {
  static constexpr int NT = TS == 64 ? 256 : 512, NW = NT / 64, WN = NW / 2;
  static constexpr int TM = TS / 2, TN = TS / WN;   // a wave's tile
  static constexpr int FM = TM / 16, FN = TN / 16;  // in 16 x 16 matrix tiles
  static constexpr int SUMS_OFF = 0;
};
template <int TS, bool W4, RowKind KIND, int EPI>
__global__ __launch_bounds__(AnyCfg<TS>::NT, TS == 64 ? 4 : 2) void qgemm_any(
    const int8_t* __restrict__ A, const void* __restrict__ Wv, int64_t M, int64_t N, int64_t K,
    const float* __restrict__ a_scale, const float* __restrict__ w_scale, int w_per_row, float* __restrict__ Y,
    int32_t* __restrict__ ACC, EpiArgs epi) {
  using C = AnyCfg<TS>;
  using SA = AnyStage<C::NT, TS, 8, KIND>;
  using SB = AnyStage<C::NT, TS, W4 ? 4 : 8, KIND>;
  constexpr bool SHORT = KIND == kRowsShort;
  __shared__ __attribute__((aligned(16))) int8_t lds_a[2][TS * kAnyBK];
  __shared__ __attribute__((aligned(16))) int8_t lds_b[2][TS * kAnyBK];
  __shared__ __attribute__((aligned(16))) float scales[TS];
  __shared__ float sums[C::NW];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wm = wave / C::WN, wn = wave % C::WN;
  const int64_t m0 = (int64_t)blockIdx.y * TS, n0 = (int64_t)blockIdx.x * TS;

  SA sa_;
  SB sb_;
  sa_.init(A, M, K, m0);
  sb_.init(Wv, N, W4 ? K >> 1 : K, n0);
  constexpr int BKB = W4 ? kAnyBK / 2 : kAnyBK;  // bytes of k per W tile row in memory
  constexpr int NS = SHORT ? 1 : 3;
  v4i ra[NS][SA::CN], rb[NS][SB::CN];  // k tiles t, t + 1 and t + 2; tile KT, behind the last one, ends it
  const int KT = SHORT ? 1 : (int)((K + kAnyBK - 1) / kAnyBK);
#pragma unroll
  for (int u = 0; u < NS; ++u) {
    sa_.load(ra[u], u * kAnyBK);
    sb_.load(rb[u], u * BKB);
  }
  const bool want_y = EPI != 0 || Y != nullptr;
  const float sa = f_from_bits(__builtin_amdgcn_readfirstlane(bits_from_f(want_y ? a_scale[0] : 0.0f)));
  if (want_y && (int)threadIdx.x < TS) {
    const int64_t n = n0 + (int)threadIdx.x;
    scales[threadIdx.x] = w_scale[w_per_row && n < N ? n : 0];
  }
  float q_inv = 0.0f, q_max = 0.0f;
  if (EPI == 3) {
    float q_scale;
    bit_constants(epi.q_absmax[0], epi.q_bits, q_scale, q_inv);
    q_max = (float)((1 << (epi.q_bits - 1)) - 1);
  }
  v4i acc[C::FM][C::FN];
  zero_acc(acc);
  for (int kt = 0; kt < KT; kt += NS) {
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const int t = kt + u, next = (u + 1) % NS;
      if (t >= KT) break;  // workgroup-uniform
      // this buffer was last read in step t - 2; every wave has passed the barrier of step t - 1 since
      int8_t* la = lds_a[t & 1];
      int8_t* lb = lds_b[t & 1];
      auto store = [&](auto edge) {
        constexpr bool EDGE = decltype(edge)::value;
        store8<EDGE>(la, sa_, ra[u], ra[next], t * kAnyBK);
        if constexpr (W4) store4<EDGE>(lb, sb_, rb[u], rb[next], t * BKB);
        else store8<EDGE>(lb, sb_, rb[u], rb[next], t * BKB);
      };
      if (!SHORT && sa_.edge(t * kAnyBK)) store(std::true_type{});  // (both operands end in the same k tile)
      else store(std::false_type{});
      if (!SHORT) {  // past the row's end, where loads stay at its last bytes, as well: under a condition the compiler would
        // take it as not issued and wait for the tile before it
        sa_.load(ra[u], (t + NS) * kAnyBK);
        sb_.load(rb[u], (t + NS) * BKB);
      }
      __syncthreads();
      v4i fa[2][C::FM], fb[2][C::FN];
#pragma unroll
      for (int s = 0; s < 2; ++s) {  // 64 k each
        const int ch = 4 * s + (lane >> 4);
#pragma unroll
        for (int j = 0; j < C::FN; ++j)
          fb[s][j] = *reinterpret_cast<const v4i*>(lb + lds_off(wn * C::TN + j * 16 + (lane & 15), ch));
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
          fa[s][i] = *reinterpret_cast<const v4i*>(la + lds_off(wm * C::TM + i * 16 + (lane & 15), ch));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < C::FN; ++j)
#pragma unroll
          for (int i = 0; i < C::FM; ++i) mma(acc[i][j], fb[s][j], fa[s][i]);
    }
  }
  acc_ready(acc);
  float sse = 0.0f, amax = 0.0f;
  epilogue<C, W4, false, EPI>(acc, m0, n0, wm, wn, lane, reinterpret_cast<const char*>(scales), M, N, sa, want_y, q_inv, q_max, Y,
                              ACC, epi, sse, amax);
  finish_sums<C, EPI>(reinterpret_cast<char*>(sums), wave, sse, amax, epi, (int64_t)blockIdx.y * gridDim.x + blockIdx.x);
}

// sum of `count` per-workgroup partials, one workgroup, fixed order
__global__ __launch_bounds__(kBlock) void sum_partials_k(const double* __restrict__ part, int64_t count,
                                                         double* __restrict__ out) {
  __shared__ double sm[kBlock];
  double a = 0.0;
  for (int64_t i = threadIdx.x; i < count; i += kBlock) a += part[i];
  sm[threadIdx.x] = a;
  __syncthreads();
  for (int h = kBlock / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) sm[threadIdx.x] += sm[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = sm[0];
}


// ---- split along k ----------------------------------------------------------------------------------
// A GEMM with a few dozen output tiles and a long k (512 x 4608 x 512 is 64 tiles of 64 x 64) leaves most of
// the chip idle.  With a workspace the caller lets the library cut k into `split` ranges: every (tile,
// range) pair is a workgroup that writes its raw int32 accumulators to a plane of the workspace, and
// one elementwise kernel adds the planes (integer sums: exact in any order, so the accumulators stay
// bit-identical to the unsplit product) and applies the epilogue Y = (float(acc) * s_A) * s_W[n].
// Layers of at most one or two 16 x 16 tiles per CU come here with a long k only (split_beats_skinny).
// Measured on the chip: the second kernel and the planes cost about 5 us, so the split pays only
// where the unsplit grid is tiny; 1568 x 4608 x 512 (200 tiles of 64 x 64: 17 us) and 6272 x 2304 x 256
// (14.6 us) lose 5-9 us with any split of either tile size, and stay unsplit.
struct SplitPlan {
  int split = 1;
  int k_per_split = 0;
};

static SplitPlan plan_split(int64_t M, int64_t N, int64_t K) {
  SplitPlan p;
  const int64_t base = ((M + 63) / 64) * ((N + 63) / 64);  // tiles of 64 x 64
  if (K < 1024 || base > kNumCU / 4) return p;
  const int64_t kt = (K + 127) / 128;               // k tiles of 128 bytes
  int64_t want = (kNumCU + base - 1) / base;        // about one workgroup per CU
  if (want > 16) want = 16;
  if (want > kt / 2) want = kt / 2;                 // at least two k tiles per range
  if (want < 2) return p;
  const int64_t per = (kt + want - 1) / want;       // k tiles per range
  p.k_per_split = (int)(per * 128);
  p.split = (int)((kt + per - 1) / per);            // no empty range
  if (p.split < 2) return SplitPlan{};
  return p;
}

// Layers that qgemm_skinny could take as well: with a workspace the split wins once k is long.  us, split | skinny
// (M x N, int8 next to packed int4): 16 x 256 K = 8192 10.3 | 9.8 next to 10.8 | 8.1, 12288 10.4 | 13.2 next to
// 10.7 | 10.7, 32768 13.5 | 30.7 next to 14.6 | 23.7; 128 x 512 K = 8192 11.8 | 10.2, 12288 12.0 | 13.9 next to 12.2 | 11.1,
// 16384 12.8 | 17.8 next to 13.3 | 13.8; 16 x 4096, cut in four only, K = 12288 13.9 | 15.0, 32768 25.6 | 38.5 next to 28 | 25;
// 1 x 1024, whose A is one row, packed int4 K = 16384 11.7 | 8.9, 32768 14.7 | 15.1.
static bool split_beats_skinny(const SplitPlan& p, int64_t M, int64_t K, bool w4) {
  if (w4) return K > (M == 1 ? 28672 : 13312) && p.split >= 8;
  return K > 9216;
}

// acc = sum of `split` planes; ACC and / or Y from it.  VEC: four consecutive n per thread.
template <bool VEC>
__global__ __launch_bounds__(kBlock) void splitk_reduce(const int32_t* __restrict__ planes, int split, int64_t MN,
                                                        int64_t N, const float* __restrict__ a_scale,
                                                        const float* __restrict__ w_scale, int w_per_row,
                                                        float* __restrict__ Y, int32_t* __restrict__ ACC) {
  const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * (VEC ? 4 : 1);
  if (i >= MN) return;
  const float sa = Y ? a_scale[0] : 0.0f;
  if (VEC) {
    v4i a = *reinterpret_cast<const v4i*>(planes + i);
    for (int s = 1; s < split; ++s) {
      const v4i b = *reinterpret_cast<const v4i*>(planes + (int64_t)s * MN + i);
      a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    if (ACC) *reinterpret_cast<v4i*>(ACC + i) = a;
    if (Y) {
      const int64_t n = i % N;  // N % 4 == 0: the four share a row
      float4 sw;
      if (w_per_row) sw = *reinterpret_cast<const float4*>(w_scale + n);
      else sw = make_float4(w_scale[0], w_scale[0], w_scale[0], w_scale[0]);
      *reinterpret_cast<float4*>(Y + i) = make_float4(((float)a.x * sa) * sw.x, ((float)a.y * sa) * sw.y,
                                                      ((float)a.z * sa) * sw.z, ((float)a.w * sa) * sw.w);
    }
  } else {
    int a = planes[i];
    for (int s = 1; s < split; ++s) a += planes[(int64_t)s * MN + i];
    if (ACC) ACC[i] = a;
    if (Y) Y[i] = ((float)a * sa) * w_scale[w_per_row ? i % N : 0];
  }
}

// Everything about the arguments of a quantized layer that can be wrong, checked on the host
// before anything is enqueued (a failing call leaves the device untouched).
static int check_qgemm_args(const int8_t* a_q, const void* w_q, int w_storage_bits, int64_t M, int64_t N, int64_t K,
                            const float* a_scale, const float* w_scale, int w_gran, const float* y_out,
                            const int32_t* acc_out, const EpiArgs& epi) {
  const float* y_ref = epi.yref;
  if (!a_q || !w_q) return MPQ_ERR_NULL;
  if (!y_out && !acc_out && !y_ref && !epi.amax && !epi.codes) return MPQ_ERR_NULL;
  if ((y_out || y_ref || epi.amax || epi.codes) && (!a_scale || !w_scale)) return MPQ_ERR_NULL;
  if (w_storage_bits != 8 && w_storage_bits != 4) return MPQ_ERR_BITS;
  if (M <= 0 || N <= 0 || K <= 0) return MPQ_ERR_SHAPE;
  if (K > 133143) return MPQ_ERR_SHAPE;  // K * 127 * 127 must stay below 2^31
  if (w_storage_bits == 4 && (K & 1)) return MPQ_ERR_SHAPE;
  if (mul_overflows(M, N) || mul_overflows(M, K) || mul_overflows(N, K)) return MPQ_ERR_SHAPE;
  if (w_gran != MPQ_PER_TENSOR && w_gran != MPQ_PER_ROW) return MPQ_ERR_GRAN;
  if (y_out && (reinterpret_cast<uintptr_t>(y_out) & 3u)) return MPQ_ERR_ALIGN;
  if (y_ref && (reinterpret_cast<uintptr_t>(y_ref) & 3u)) return MPQ_ERR_ALIGN;
  if (acc_out && (reinterpret_cast<uintptr_t>(acc_out) & 3u)) return MPQ_ERR_ALIGN;
  const int64_t gx = (N + 127) / 128, gy = (M + 127) / 128;
  if (gx > 0x7FFFFFFF || gy > kMaxGridY) return MPQ_ERR_SHAPE;       // grid of qgemm_any (see any_tile)
  if (((M + 63) / 64) * ((N + 63) / 64) > 0x7FFFFFFF) return MPQ_ERR_SHAPE;  // ... and of the smallest fast tile
  return MPQ_OK;
}

static bool fast_path(const int8_t* a_q, const void* w_q, bool w4, int64_t M, int64_t N, int64_t K) {
  // the fast kernels index rows with 32 bits
  return aligned16(a_q) && aligned16(w_q) && (K % (w4 ? 32 : 16)) == 0 && M < (1ll << 31) && N < (1ll << 31);
}

// Dispatch shared by every quantized-layer call; the arguments have passed check_qgemm_args.  With
// y_ref the kernels also leave one partial sum of (Y - y_ref)^2 per workgroup in epi.part and
// report how many.  ws / ws_bytes: optional scratch for the split along k (plain epilogue only).
static int run_qgemm(const int8_t* a_q, const void* w_q, int w_storage_bits, int64_t M, int64_t N,
                     int64_t K, const float* a_scale, const float* w_scale, int w_gran, float* y_out,
                     int32_t* acc_out, EpiArgs epi, int64_t* n_partials, hipStream_t st, void* ws = nullptr,
                     size_t ws_bytes = 0) {
  const int per_row = w_gran == MPQ_PER_ROW;
  const bool w4 = w_storage_bits == 4;
  // (the score keeps one partial per 64 x 64 tile at most: its workspace holds no more)
  const bool fast = fast_path(a_q, w_q, w4, M, N, K);
  const int waves = epi.yref ? 0 : skinny_waves(M, N, K, fast && epi.amax);
  const bool plain = !epi.yref && !epi.codes && !epi.act && !epi.amax;
  const SplitPlan sp = plain && fast ? plan_split(M, N, K) : SplitPlan{};
  const bool split = sp.split > 1 && ws && aligned16(ws) && ws_bytes >= (size_t)sp.split * (size_t)(M * N) * sizeof(int32_t);
  if (waves && !(split && split_beats_skinny(sp, M, K, w4)))
    return launch_skinny(waves, w4, DmaArgs{a_q, w_q, M, N, K, a_scale, w_scale, per_row, y_out, acc_out, st, epi,
                                            n_partials, 1, 0, false});
  if (fast) {
    DmaArgs d{a_q, w_q, M, N, K, a_scale, w_scale, per_row, y_out, acc_out, st, epi, n_partials, 1, 0, false};
    if (split) {
      int32_t* planes = reinterpret_cast<int32_t*>(ws);
      d.y_out = nullptr;
      d.acc_out = planes;
      d.split = sp.split;
      d.k_per_split = sp.k_per_split;
      const int rc = launch_dma_64(w4, 3, 128, d);
      if (rc != MPQ_OK) return rc;
      const int64_t MN = M * N;
      const bool vec = (N & 3) == 0 && (!y_out || aligned16(y_out)) && (!acc_out || aligned16(acc_out)) &&
                       (!(y_out && per_row) || aligned16(w_scale));
      const int64_t threads = vec ? MN / 4 : MN;
      const unsigned blocks = (unsigned)((threads + kBlock - 1) / kBlock);
      if (vec) splitk_reduce<true><<<blocks, kBlock, 0, st>>>(planes, sp.split, MN, N, a_scale, w_scale, per_row, y_out, acc_out);
      else splitk_reduce<false><<<blocks, kBlock, 0, st>>>(planes, sp.split, MN, N, a_scale, w_scale, per_row, y_out, acc_out);
      return launch_status();
    }
    const FastTile t = fast_tile(M, N, K, kNumCU);
    if (t.side == 256) return launch_dma_256(w4, d);
    if (t.side == 192) return launch_dma_192(w4, t.stages, d);
    if (t.side == 128) return launch_dma_128(w4, t.stages, d);
    return launch_dma_64(w4, t.stages, t.kb, d);
  }
  const int ts = any_tile(M, N, K, kNumCU);
  const int64_t gx = (N + ts - 1) / ts, gy = (M + ts - 1) / ts;
  const dim3 grid((unsigned)gx, (unsigned)gy);
  const int64_t w_row = w4 ? K >> 1 : K;
  const bool dword = ((K | w_row | (int64_t)reinterpret_cast<uintptr_t>(a_q) | (int64_t)reinterpret_cast<uintptr_t>(w_q)) & 3) == 0;
  const RowKind kind = w_row < 16 ? kRowsShort : dword ? kRowsDword : kRowsByte;
  const int mode = epi.yref ? 1 : epi.codes ? 3 : (epi.act || epi.amax) ? 2 : 0;
#define MPQ_ANY(TS_, W4_, KIND_, EPI_)                                                                                    \
  qgemm_any<TS_, W4_, KIND_, EPI_><<<grid, AnyCfg<TS_>::NT, 0, st>>>(a_q, w_q, M, N, K, a_scale, w_scale, per_row, y_out, \
                                                                     acc_out, epi)
#define MPQ_ANY_EPI(TS_, W4_, KIND_)               \
  (mode == 1   ? (void)MPQ_ANY(TS_, W4_, KIND_, 1) \
   : mode == 2 ? (void)MPQ_ANY(TS_, W4_, KIND_, 2) \
   : mode == 3 ? (void)MPQ_ANY(TS_, W4_, KIND_, 3) \
               : (void)MPQ_ANY(TS_, W4_, KIND_, 0))
#define MPQ_ANY_KIND(TS_, W4_)                                      \
  (kind == kRowsShort   ? MPQ_ANY_EPI(TS_, W4_, kRowsShort)         \
   : kind == kRowsDword ? MPQ_ANY_EPI(TS_, W4_, kRowsDword)         \
                        : MPQ_ANY_EPI(TS_, W4_, kRowsByte))
  if (ts == 128) {
    if (w4) MPQ_ANY_KIND(128, true);
    else MPQ_ANY_KIND(128, false);
  } else {
    if (w4) MPQ_ANY_KIND(64, true);
    else MPQ_ANY_KIND(64, false);
  }
#undef MPQ_ANY_KIND
#undef MPQ_ANY_EPI
#undef MPQ_ANY
  if (n_partials) *n_partials = gx * gy;
  return launch_status();
}

// partials never outnumber the 64 x 64 tiles (the smallest tile any kernel here uses)
static int64_t max_partials(int64_t M, int64_t N) { return ((M + 63) / 64) * ((N + 63) / 64); }

}  // namespace mpq

using namespace mpq;

extern "C" int mpq_init(void) {
  const DmaArgs d{nullptr, nullptr, 0, 0, 0, nullptr, nullptr, 0, nullptr, nullptr, nullptr, kNoEpi, nullptr, 1, 0, true};
  for (int w4 = 0; w4 < 2; ++w4) {
    int rc = launch_dma_256(w4 != 0, d);
    for (int stages = 2; stages <= 3; ++stages) {
      if (rc == MPQ_OK) rc = launch_dma_192(w4 != 0, stages, d);
      if (rc == MPQ_OK) rc = launch_dma_128(w4 != 0, stages, d);
      for (int kb = 128; kb <= 256; kb += 128)
        if (rc == MPQ_OK) rc = launch_dma_64(w4 != 0, stages, kb, d);
    }
    if (rc != MPQ_OK) return rc;
  }
  return prepare_hutchinson();
}

extern "C" size_t mpq_qgemm_workspace_bytes(int64_t M, int64_t N, int64_t K, int w_storage_bits) {
  if (M <= 0 || N <= 0 || K <= 0 || K > 133143 || (w_storage_bits != 8 && w_storage_bits != 4)) return 0;
  if (mul_overflows(M, N) || mul_overflows(M, K) || mul_overflows(N, K)) return 0;
  const SplitPlan sp = plan_split(M, N, K);
  return sp.split > 1 ? (size_t)sp.split * (size_t)(M * N) * sizeof(int32_t) : 0;
}

extern "C" int mpq_qgemm(const int8_t* a_q, const void* w_q, int w_storage_bits, int64_t M,
                         int64_t N, int64_t K, const float* a_scale, const float* w_scale,
                         int w_gran, float* y_out, int32_t* acc_out, void* ws, size_t ws_bytes,
                         void* stream) {
  if (!y_out && !acc_out) return MPQ_ERR_NULL;
  const int rc = check_qgemm_args(a_q, w_q, w_storage_bits, M, N, K, a_scale, w_scale, w_gran, y_out, acc_out, kNoEpi);
  if (rc != MPQ_OK) return rc;
  return run_qgemm(a_q, w_q, w_storage_bits, M, N, K, a_scale, w_scale, w_gran, y_out, acc_out,
                   kNoEpi, nullptr, (hipStream_t)stream, ws, ws_bytes);
}

// shared by mpq_qgemm_act and mpq_stack_evaluate (which checks all its layers before its first launch)
namespace mpq {
int check_qgemm_act_args(const int8_t* a_q, const void* w_q, int w_storage_bits, int64_t M, int64_t N, int64_t K,
                         const float* a_scale, const float* w_scale, int w_gran, int act, const float* y_out,
                         const float* absmax_out) {
  if (!y_out && !absmax_out) return MPQ_ERR_NULL;
  if (act < MPQ_ACT_NONE || act > MPQ_ACT_GELU) return MPQ_ERR_SHAPE;
  if (absmax_out && (reinterpret_cast<uintptr_t>(absmax_out) & 3u)) return MPQ_ERR_ALIGN;
  const EpiArgs epi{nullptr, nullptr, act, reinterpret_cast<unsigned*>(const_cast<float*>(absmax_out)), nullptr, 0, nullptr};
  return check_qgemm_args(a_q, w_q, w_storage_bits, M, N, K, a_scale, w_scale, w_gran, y_out, nullptr, epi);
}
int check_qgemm_score_args(const int8_t* a_q, const void* w_q, int w_storage_bits, int64_t M, int64_t N, int64_t K,
                           const float* a_scale, const float* w_scale, int w_gran, const float* y_ref,
                           const double* sse_out, const float* y_out, const void* ws, size_t ws_bytes) {
  if (!y_ref || !sse_out) return MPQ_ERR_NULL;
  if (reinterpret_cast<uintptr_t>(sse_out) & 7u) return MPQ_ERR_ALIGN;
  if (M <= 0 || N <= 0 || mul_overflows(M, N)) return MPQ_ERR_SHAPE;
  if (!ws || ws_bytes < (size_t)max_partials(M, N) * sizeof(double)) return MPQ_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(ws) & 7u) return MPQ_ERR_ALIGN;
  const EpiArgs epi{y_ref, nullptr, 0, nullptr, nullptr, 0, nullptr};
  return check_qgemm_args(a_q, w_q, w_storage_bits, M, N, K, a_scale, w_scale, w_gran, y_out, nullptr, epi);
}
}  // namespace mpq

// mpq_qgemm_act for mpq_stack_evaluate, arguments already checked: the running maximum goes to `part` as one
// value per workgroup, their number to *parts, where the layer takes the tiled kernels and there are at most
// `room` of them; else *parts = 0 and the maximum is merged into absmax_out as usual.
namespace mpq {
int qgemm_act_partials(const int8_t* a_q, const void* w_q, int w_storage_bits, int64_t M, int64_t N, int64_t K,
                       const float* a_scale, const float* w_scale, int w_gran, int act, float* y_out,
                       float* absmax_out, float* part, int64_t room, int* parts, hipStream_t st) {
  EpiArgs epi{nullptr, nullptr, act, reinterpret_cast<unsigned*>(absmax_out), nullptr, 0, nullptr};
  *parts = 0;
  const bool tiled = fast_path(a_q, w_q, w_storage_bits == 4, M, N, K) && !skinny_waves(M, N, K, true);
  int64_t count = 0;
  if (tiled && max_partials(M, N) <= room) epi.amax_part = part;
  const int rc = run_qgemm(a_q, w_q, w_storage_bits, M, N, K, a_scale, w_scale, w_gran, y_out, nullptr, epi, &count, st);
  if (epi.amax_part) *parts = (int)count;
  return rc;
}
}  // namespace mpq

extern "C" int mpq_qgemm_act(const int8_t* a_q, const void* w_q, int w_storage_bits, int64_t M, int64_t N,
                             int64_t K, const float* a_scale, const float* w_scale, int w_gran, int act,
                             float* y_out, float* absmax_out, int accumulate, void* stream) {
  // every check comes before the fill: a failing call leaves the device untouched
  const int rc = check_qgemm_act_args(a_q, w_q, w_storage_bits, M, N, K, a_scale, w_scale, w_gran, act, y_out, absmax_out);
  if (rc != MPQ_OK) return rc;
  hipStream_t st = (hipStream_t)stream;
  unsigned* amax = reinterpret_cast<unsigned*>(absmax_out);
  if (amax && !accumulate) fill_u32_k<<<1, 1, 0, st>>>(amax, 0u);
  return run_qgemm(a_q, w_q, w_storage_bits, M, N, K, a_scale, w_scale, w_gran, y_out, nullptr,
                   EpiArgs{nullptr, nullptr, act, amax, nullptr, 0, nullptr}, nullptr, st);
}

extern "C" int mpq_qgemm_act_codes(const int8_t* a_q, const void* w_q, int w_storage_bits, int64_t M, int64_t N,
                                   int64_t K, const float* a_scale, const float* w_scale, int w_gran, int act,
                                   const float* absmax, int bits, int8_t* codes_out, void* stream) {
  if (!absmax || !codes_out) return MPQ_ERR_NULL;
  if (act < MPQ_ACT_NONE || act > MPQ_ACT_GELU) return MPQ_ERR_SHAPE;
  if (bits < 2 || bits > 8) return MPQ_ERR_BITS;
  if (reinterpret_cast<uintptr_t>(absmax) & 3u) return MPQ_ERR_ALIGN;
  const EpiArgs epi{nullptr, nullptr, act, nullptr, absmax, bits, codes_out};
  const int rc = check_qgemm_args(a_q, w_q, w_storage_bits, M, N, K, a_scale, w_scale, w_gran, nullptr, nullptr, epi);
  if (rc != MPQ_OK) return rc;
  return run_qgemm(a_q, w_q, w_storage_bits, M, N, K, a_scale, w_scale, w_gran, nullptr, nullptr, epi, nullptr,
                   (hipStream_t)stream);
}

extern "C" size_t mpq_qgemm_score_workspace_bytes(int64_t M, int64_t N, int64_t K, int w_storage_bits) {
  (void)w_storage_bits;
  if (M <= 0 || N <= 0 || K <= 0 || mul_overflows(M, N)) return 0;
  return (size_t)max_partials(M, N) * sizeof(double);
}

extern "C" int mpq_qgemm_score(const int8_t* a_q, const void* w_q, int w_storage_bits, int64_t M,
                               int64_t N, int64_t K, const float* a_scale, const float* w_scale,
                               int w_gran, const float* y_ref, double* sse_out, float* y_out, void* ws,
                               size_t ws_bytes, void* stream) {
  int rc = check_qgemm_score_args(a_q, w_q, w_storage_bits, M, N, K, a_scale, w_scale, w_gran, y_ref, sse_out, y_out, ws,
                                  ws_bytes);
  if (rc != MPQ_OK) return rc;
  hipStream_t st = (hipStream_t)stream;
  double* partials = reinterpret_cast<double*>(ws);
  int64_t count = 0;
  rc = run_qgemm(a_q, w_q, w_storage_bits, M, N, K, a_scale, w_scale, w_gran, y_out, nullptr,
                 EpiArgs{y_ref, partials, 0, nullptr, nullptr, 0, nullptr}, &count, st);
  if (rc != MPQ_OK) return rc;
  sum_partials_k<<<1, kBlock, 0, st>>>(partials, count, sse_out);
  return launch_status();
}
