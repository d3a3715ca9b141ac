// qgemm_quad.hpp -- the large tiles of the quantized linear layer's fast path: qgemm_dma.hpp's global->LDS
// pipeline with every k tile taken in four quarters.
//
// Each wave's tile is cut in two along M (A halves 0, 1) and in two along N (W halves 0, 1), and a k tile of
// 128 is multiplied as A0 W0, A0 W1, A1 W1, A1 W0.  Each quarter brings exactly one new half into registers, and
// that half is read from LDS a quarter ahead:
//   quarter 0  A0 W0   reads W1 of this k tile
//   quarter 1  A0 W1   reads A1
//   quarter 2  A1 W1   reads A0 of the next k tile
//   quarter 3  A1 W0   reads W0 of the next k tile, into the registers of W1 (so the two W register sets
//                      change places with every k tile)
// A half's place in LDS is free as soon as it has been read, long before the whole stage is, so the requests for the
// k tile NSTAGE further on go out half by half: after the barrier in front of quarter 0 for A0 and W0,
// after the one in front of quarter 2 for A1 and W1.  They are spread evenly over the k tile and each has
// NSTAGE - 1/2 k tiles of time to arrive.
//
// (The other tiles keep their waves' operands of 64 k in registers twice over; here the accumulators take half of them.)
//
// What bounds it: with int8 weights a k tile takes a CU 1.36 us (16384 x 4096 x 1024, one output tile per CU), of which
// the matrix steps alone are 1.05-1.17; at 2.0 GHz 2900 clocks passed for 2048 of matrix steps when it took 1.43.  Then,
// without its requests it took 1.05, without its LDS reads 1.33, without barriers and waits 1.33: the loads into the
// LDS, and the power they take, are what is left, and where in the k tile they are issued makes no difference (spread,
// bunched, the two waves of a SIMD apart).  A further output tile costs 10 us besides (the same
// k tiles as four output tiles per workgroup, 16384 x 1024 x 4096, 91.0 us against 61.6): its 256 KiB at the memory's rate.
// Against a barrier per k tile, a whole stage freed at once and 32x32 matrix steps: 16384 x 4096 x 1024 67.8 -> 57.9 us
// (packed weights 71.2 -> 60.5), 4096 x 4096 x 4096 67.5 -> 58.2, 16384 x 1024 x 4096 100.4 -> 91.3 (99.0 -> 87.3).
#pragma once

#include "qgemm_dma.hpp"

namespace mpq {

template <class C, int BM, int BN, bool W4>
struct QuadPlan {
  static constexpr int TMH = C::TM / 2, TNH = C::TN / 2;     // a wave's rows of one half
  static constexpr int NA = BM / 2 / C::RPI / C::NW;      // wave-loads per wave of an A half
  static constexpr int BRPI = W4 ? C::PRPI : C::RPI;
  static constexpr int NB = BN / 2 / BRPI / C::NW;        // ... and of a W half
  static_assert(NA * C::RPI * C::NW * 2 == BM && NB * BRPI * C::NW * 2 == BN, "loads divide evenly over the waves");
  static_assert(C::DBK == 128 && NA <= 2 && NB <= 2, "k tile of 128, at most two wave-loads per half");
  // wave-load r of wave w covers rows (w * N + r) * RPI ... of a half; those lie in the rows of one wave's tile
  static_assert(TMH % (NA * C::RPI) == 0 && TNH % (NB * BRPI) == 0, "a wave's loads of a half stay in one wave's rows");

  unsigned off_a[2][NA], off_b[2][NB];  // bytes from the tile's first row (k = 0) for half h, load r
  unsigned lds_a, lds_b;                // LDS offset of the wave's first row of half 0, load 0
  unsigned ka, kb;                      // the lane's k within a tile (load 0; load 1 differs by KX1)
  static constexpr unsigned KX1 = 64;   // its rows start 8 further on, which flips one bit of the swizzle

  __device__ __forceinline__ static int row_a(int wave) { return wave * NA * C::RPI / TMH * C::TM + wave * NA * C::RPI % TMH; }
  __device__ __forceinline__ static int row_b(int wave) { return wave * NB * BRPI / TNH * C::TN + wave * NB * BRPI % TNH; }

  __device__ __forceinline__ void init(int wave, int lane) {
    lds_a = (unsigned)(row_a(wave) * C::DBK);
    lds_b = (unsigned)(C::A_STAGE + row_b(wave) * C::B_ROW);
    // logical chunk of the lane: LDS slot ^ row swizzle (int8: (row >> 1) & 7, packed: (row >> 2) & 3)
    ka = (unsigned)(((lane & 7) ^ ((lane >> 4) & 3) ^ ((row_a(wave) >> 1) & 4)) * 16);
    kb = W4 ? (unsigned)(((lane & 3) ^ ((lane >> 4) & 3)) * 32) : (unsigned)(((lane & 7) ^ ((lane >> 4) & 3) ^ ((row_b(wave) >> 1) & 4)) * 16);
  }
  // rows past the edge re-read the last row; never stored.  last: last valid row, counted from the tile's first
  __device__ __forceinline__ void rows_a(int wave, int lane, unsigned K, unsigned last) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < NA; ++r) {
        unsigned row = (unsigned)(row_a(wave) + h * TMH + r * C::RPI + (lane >> 3));
        row = row < last ? row : last;
        off_a[h][r] = row * K + (r ? ka ^ KX1 : ka);
      }
  }
  __device__ __forceinline__ void rows_b(int wave, int lane, unsigned K, unsigned last) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < NB; ++r) {
        unsigned row = (unsigned)(row_b(wave) + h * TNH + r * BRPI + (W4 ? lane >> 2 : lane >> 3));
        row = row < last ? row : last;
        off_b[h][r] = W4 ? row * (K >> 1) + (kb >> 1) : row * K + (r ? kb ^ KX1 : kb);
      }
  }
};

// Grid, chunks and options as qgemm_dma; k in tiles of 128, any number of them.
template <int BM, int BN, int WM, int WN, int NSTAGE, bool W4, bool VEC, int EPI>
__global__ __launch_bounds__(WM * WN * 64, 1) void qgemm_quad(const int8_t* __restrict__ A, const void* __restrict__ Wv,
                                                             int64_t M, int64_t N, int64_t K,
                                                             const float* __restrict__ a_scale,
                                                             const float* __restrict__ w_scale, int w_per_row,
                                                             float* __restrict__ Y, int32_t* __restrict__ ACC, EpiArgs epi,
                                                             int tiles_n, int tiles_m, int chunk, int remap) {
  constexpr bool QOUT = EPI == 3;
  using C = DmaCfg<BM, BN, WM, WN, NSTAGE, W4, 128>;
  using P = QuadPlan<C, BM, BN, W4>;
  constexpr int HM = C::FM / 2, HN = C::FN / 2;  // 16x16 tiles of a half
  static_assert(C::FM % 2 == 0 && C::FN % 2 == 0, "halves of whole 16x16 tiles");
  constexpr int LH = P::NA + P::NB;              // a wave's requests per half k tile
  constexpr int WAIT = (NSTAGE - 1) * 2 * LH;    // ... issued after the ones a barrier waits for
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wm = wave / WN, wn = wave % WN;
  const unsigned lds0 = (unsigned)(uintptr_t)MPQ_LPTR(lds);
  const int G = (int)gridDim.x;
  int wg = (int)blockIdx.x;
  if (remap) wg = (wg & 7) * (G >> 3) + (wg >> 3);  // G % 8 == 0
  const int KT = (int)((K + 127) >> 7);
  const unsigned Ku = (unsigned)K;
  int tile = (wg / tiles_n) * chunk;
  const int tile_end = tile + chunk < tiles_m ? tile + chunk : tiles_m;
  const int64_t n0 = (int64_t)(wg % tiles_n) * BN;
  const bool want_y = EPI != 0 || Y != nullptr;

  P plan;
  plan.init(wave, lane);
  plan.rows_b(wave, lane, Ku, (unsigned)(N - 1 - n0 < BN ? N - 1 - n0 : BN));
  const char* const b_first = reinterpret_cast<const char*>(Wv) + n0 * (W4 ? K >> 1 : K);
  Cursor<128, W4> cursor;
  cursor.init(nullptr, b_first, (int)K, tile);
  auto start_rows = [&](bool first) {  // see qgemm_dma
    const int64_t m = (int64_t)cursor.tile * BM;
    cursor.a = reinterpret_cast<const char*>(A) + m * K;
    cursor.b = b_first;
    if (first || m + BM > M) plan.rows_a(wave, first ? lane : lane_again(), Ku, (unsigned)(M - 1 - m < BM ? M - 1 - m : BM));
  };
  start_rows(true);
  // request r (A loads first) of half h of the cursor's k tile into the stage at LDS offset `stage`
  auto request = [&](auto whole_, auto h_, auto r_, unsigned stage) {
    constexpr bool WHOLE = decltype(whole_)::value;
    constexpr int h = decltype(h_)::value, r = decltype(r_)::value;
    if constexpr (r < P::NA) {
      cursor.template fetch<WHOLE, true>(plan.off_a[h][r], r ? plan.ka ^ P::KX1 : plan.ka,
                                  lds0 + stage + plan.lds_a + (unsigned)((h * P::TMH + r * C::RPI) * C::DBK));
    } else {
      constexpr int x = r - P::NA;
      cursor.template fetch<WHOLE, false>(plan.off_b[h][x], !W4 && x ? plan.kb ^ P::KX1 : plan.kb,
                                   lds0 + stage + plan.lds_b + (unsigned)((h * P::TNH + x * P::BRPI) * C::B_ROW));
    }
  };
  if (want_y && w_per_row) request_scales<VEC>(w_scale, n0, N, BN, lane, lds0 + C::SCALE_OFF);
#pragma unroll 1
  for (int p = 0; p < NSTAGE; ++p) {
    auto both = [&](auto whole_) {
      static_for<0, LH>([&](auto r_) { request(whole_, std::integral_constant<int, 0>{}, r_, (unsigned)(p * C::STAGE)); });
      static_for<0, LH>([&](auto r_) { request(whole_, std::integral_constant<int, 1>{}, r_, (unsigned)(p * C::STAGE)); });
    };
    if (cursor.whole()) both(std::true_type{});
    else both(std::false_type{});
    if (cursor.advance(tile_end)) start_rows(false);
  }
  // the epilogue's scalars: behind the requests, into scalar registers (see qgemm_dma)
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

  // Operand registers.  fb: W4: a packed chunk serves both k halves of the tile (see FragBase).
  constexpr int BK = W4 ? 1 : 2;
  v4i fa[2][2][HM], fb[2][BK][HN];
  FragBase<C, W4> fr;
  fr.init(wm, wn, lane);
  constexpr unsigned AX = W4 ? 16 : 64;  // from the chunk of the tile's first 64 k to that of its second
  auto lds_at = [&](unsigned off) { return *reinterpret_cast<const v4i*>(lds + off); };
  // read n of an A half (2 HM of them) or a W half (BK HN)
  auto read_a = [&](auto n_, auto h_, unsigned at0, unsigned at1) {
    constexpr int n = decltype(n_)::value, h = decltype(h_)::value, ks = n / HM, i = n % HM;
    fa[h][ks][i] = lds_at((ks ? at1 : at0) + (unsigned)((h * P::TMH + i * 16) * C::DBK));
  };
  auto read_b = [&](auto n_, auto h_, auto s_, unsigned at0, unsigned at1) {
    constexpr int n = decltype(n_)::value, h = decltype(h_)::value, s = decltype(s_)::value, ks = n / HN, j = n % HN;
    fb[s][ks][j] = lds_at((ks ? at1 : at0) + (unsigned)((h * P::TNH + j * 16) * C::B_ROW));
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;

  wait_vmcnt<WAIT + LH>();  // half 0 of k tile 0
  float sse = 0.0f, amax = 0.0f;
  unsigned cur = 0;  // stage of the k tile being multiplied
  int landed = 0;    // k tiles of this output tile known to be in LDS already

  while (true) {
    lds_done();
    meet();  // see qgemm_dma
    static_for<0, 2 * HM>([&](auto n_) { read_a(n_, I0{}, fr.a + cur, (fr.a + cur) ^ AX); });
    static_for<0, BK * HN>([&](auto n_) { read_b(n_, I0{}, I0{}, fr.b + cur, (fr.b + cur) ^ 64u); });
    v4i acc[C::FM][C::FN];
    zero_acc(acc);
    // one quarter: A half HA_ (registers fa[HA_]) times W half HB_ (registers fb[SB_]); reads and requests dealt
    // out between the matrix steps
    auto quarter = [&](auto ha_, auto hb_, auto sb_, auto nread_, auto&& read, auto nreq_, auto&& req) {
      constexpr int ha = decltype(ha_)::value, hb = decltype(hb_)::value, sb = decltype(sb_)::value;
      constexpr int NR = decltype(nread_)::value, NQ = decltype(nreq_)::value;
      constexpr int NM = 2 * HM * HN;
      v4i w;
      if constexpr (W4) w = expand_half<0>(fb[sb][0][0]);
      static_for<0, NM>([&](auto m_) {
        constexpr int m = decltype(m_)::value, ks = m / (HM * HN), j = m / HM % HN, i = m % HM;
        if constexpr (!W4) w = fb[sb][W4 ? 0 : ks][j];
        mma(acc[ha * HM + i][hb * HN + j], w, fa[ha][ks][i]);
        __builtin_amdgcn_sched_barrier(0);
        static_for<m * NR * 2 / NM < NR ? m * NR * 2 / NM : NR, (m + 1) * NR * 2 / NM < NR ? (m + 1) * NR * 2 / NM : NR>(
            [&](auto n_) { read(n_); });
        static_for<m * NQ / NM, (m + 1) * NQ / NM>([&](auto r_) { req(r_); });
        if constexpr (W4 && i == HM - 1 && m + 1 < NM) {
          constexpr int m1 = m + 1, ks1 = m1 / (HM * HN), j1 = m1 / HM % HN;
          w = expand_half<ks1>(fb[sb][0][j1]);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    // k tile t; W half 0 sits in fb[S]
    auto step = [&](auto whole_, auto s_, int t) {
      constexpr int S = decltype(s_)::value;
      using Own = std::integral_constant<int, S>;
      using Other = std::integral_constant<int, S ^ 1>;
      unsigned nxt = cur + C::STAGE;
      nxt = nxt == NSTAGE * C::STAGE ? 0u : nxt;
      const unsigned a0 = fr.a + cur, b0 = fr.b + cur, an = fr.a + nxt, bn = fr.b + nxt;
      // half 1 of this k tile has landed; everyone has read half 0
      lds_done();
      if (t >= landed) wait_vmcnt<WAIT>();
      meet();
      quarter(I0{}, I0{}, Own{}, std::integral_constant<int, BK * HN>{},
              [&](auto n_) { read_b(n_, I1{}, Other{}, b0, b0 ^ 64u); }, std::integral_constant<int, P::NA>{},
              [&](auto r_) { request(whole_, I0{}, r_, cur); });
      quarter(I0{}, I1{}, Other{}, std::integral_constant<int, 2 * HM>{}, [&](auto n_) { read_a(n_, I1{}, a0, a0 ^ AX); },
              std::integral_constant<int, P::NB>{},
              [&](auto r_) { request(whole_, I0{}, std::integral_constant<int, decltype(r_)::value + P::NA>{}, cur); });
      // half 0 of the next k tile has landed; everyone has read half 1
      lds_done();
      if (t + 1 >= landed) wait_vmcnt<WAIT>();
      meet();
      quarter(I1{}, I1{}, Other{}, std::integral_constant<int, 2 * HM>{}, [&](auto n_) { read_a(n_, I0{}, an, an ^ AX); },
              std::integral_constant<int, P::NA>{}, [&](auto r_) { request(whole_, I1{}, r_, cur); });
      quarter(I1{}, I0{}, Own{}, std::integral_constant<int, BK * HN>{},
              [&](auto n_) { read_b(n_, I0{}, Other{}, bn, bn ^ 64u); }, std::integral_constant<int, P::NB>{},
              [&](auto r_) { request(whole_, I1{}, std::integral_constant<int, decltype(r_)::value + P::NA>{}, cur); });
      if (cursor.advance(tile_end)) start_rows(false);
      cur = nxt;
    };
    int t = 0;
    for (; t + 2 <= KT && cursor.whole_two(tile_end); t += 2) {
      step(std::true_type{}, I0{}, t);
      step(std::true_type{}, I1{}, t + 1);
    }
    while (t < KT) {
      step(std::false_type{}, I0{}, t);
      if (++t == KT) break;
      step(std::false_type{}, I1{}, t++);
    }
    // The next output tile's first NSTAGE k tiles land here, ahead of the stores: no wait of its first barriers
    // then has to wait for a store (both count in vmcnt).
    wait_vmcnt<0>();
    landed = NSTAGE;
    acc_ready(acc);
    epilogue<C, W4, VEC, EPI>(acc, (int64_t)tile * BM, n0, wm, wn, lane_again(), lds + C::SCALE_OFF, M, N, sa, want_y, q_inv, q_max,
                              Y, ACC, epi, sse, amax);
    if (++tile >= tile_end) break;  // block-uniform
  }
  finish_sums<C, EPI>(lds, wave, sse, amax, epi, blockIdx.x);
}

// prepare_only: configure every kernel variant of this instantiation and launch nothing (mpq_init).
template <int BM, int BN, int WM, int WN, int NSTAGE, bool W4>
static int launch_quad(const DmaArgs& a) {
  using C = DmaCfg<BM, BN, WM, WN, NSTAGE, W4, 128>;
  using Kern = void (*)(const int8_t*, const void*, int64_t, int64_t, int64_t, const float*, const float*, int,
                        float*, int32_t*, EpiArgs, int, int, int, int);
  static const Kern kerns[8] = {
      qgemm_quad<BM, BN, WM, WN, NSTAGE, W4, false, 0>, qgemm_quad<BM, BN, WM, WN, NSTAGE, W4, true, 0>,
      qgemm_quad<BM, BN, WM, WN, NSTAGE, W4, false, 1>, qgemm_quad<BM, BN, WM, WN, NSTAGE, W4, true, 1>,
      qgemm_quad<BM, BN, WM, WN, NSTAGE, W4, false, 2>, qgemm_quad<BM, BN, WM, WN, NSTAGE, W4, true, 2>,
      qgemm_quad<BM, BN, WM, WN, NSTAGE, W4, false, 3>, qgemm_quad<BM, BN, WM, WN, NSTAGE, W4, true, 3>};
  static std::atomic<unsigned> done[kMaxDevices];
  if (a.prepare_only) {
    for (int w = 0; w < 8; ++w) {
      const int rc = allow_lds(reinterpret_cast<const void*>(kerns[w]), C::LDS_BYTES, done, w);
      if (rc != MPQ_OK) return rc;
    }
    return MPQ_OK;
  }
  LaunchShape s;
  int rc = launch_shape(BM, BN, C::LDS_BYTES, a.M, a.N, a.w_scale, a.per_row, a.y_out, a.acc_out, a.epi, 1, s);
  if (rc == MPQ_OK) rc = allow_lds(reinterpret_cast<const void*>(kerns[s.which]), C::LDS_BYTES, done, s.which);
  if (rc != MPQ_OK) return rc;
  kerns[s.which]<<<(unsigned)s.grid, C::NT, C::LDS_BYTES, a.st>>>(a.a_q, a.w_q, a.M, a.N, a.K, a.a_scale, a.w_scale, a.per_row,
                                                                  a.y_out, a.acc_out, a.epi, (int)s.tn, (int)s.tm, s.chunk, s.remap);
  if (a.n_partials) *a.n_partials = s.grid;
  return launch_status();
}

}  // namespace mpq
