// Host-side selection of kernel, tile shape and epilogue for one (operand layout, operand type)
// family.  Each family is instantiated in its own translation unit to keep compile times short.
#pragma once

#include "us_gemm_direct.h"
#include "us_gemm_small.h"
#include "us_gemm_staged.h"
#include "us_launch.h"
#include <cstdlib>

namespace us {

// Tile configurations  <BM, BN, WAVES_M, WAVES_N, BKB, NST, MINB>
//   D256: 8 waves (2 x 4, 128 x 64 accumulators per wave), one workgroup per CU, 128 KB of LDS ring
//   D128: 4 waves (2 x 2, 64 x 64 per wave), two workgroups per CU, 64 KB ring
//   S128: the register-staged kernel for row pitches beyond 32-bit offsets
using CfgD256 = GemmCfg<256, 256, 2, 4, 128, 2, 1>;
//   K128: grad_W only (both operands K-strided): 8 waves on one 128 x 128 tile, two groups of 2 x 2 that
//         each take half of every 256-byte stage; one workgroup per CU, no K slices in global memory
using CfgD128 = GemmCfg<128, 128, 2, 2, 128, 2, 2>;
using CfgS128 = GemmCfg<128, 128, 2, 2, 128, 2, 2>;
using CfgK128 = GemmCfg<128, 128, 2, 2, 256, 2, 1, 2>;
//   M256: 256 x 128 tile, 8 waves as two groups of 2 x 2 sharing every stage's k-steps, three stages: FP8 outputs
//         of 192-256 such tiles (one per CU), the 512-thread shape next to K128 in a paired launch, and grad_W itself
//         (both operands K-strided) on about 128 tiles in a paired launch
using CfgM256 = GemmCfg<256, 128, 2, 2, 128, 3, 1, 2>;
//   W128: forward / grad_X with so few 128 x 128 tiles that the CUs get at most one each (BERT-base: 192): 8 waves
//         on the tile, two groups sharing the k-steps of each stage, four stages; 10-16 % faster than D128 there
using CfgW128 = GemmCfg<128, 128, 2, 2, 128, 4, 1, 2>;

//   E192: 256 x 192 tile, 8 waves (4 x 2, 64 x 96 accumulators per wave), FP16 only: outputs that make one tile per CU
//         this way and only three quarters as many 256 x 256 tiles (BERT-base: 4096 x 3072 -> 16 x 16 = 256 instead of 192)
using CfgE192 = GemmCfg<256, 192, 4, 2, 128, 2, 1>;
//   H256: 128 x 256 tile, 8 waves (2 x 4, 64 x 64 per wave): the table-driven GELU' next to grad_W tiles in a paired launch
//         whose large tiles would not fit one round
using CfgH256 = GemmCfg<128, 256, 2, 4, 128, 2, 1>;

//   Q256: 256 x 256 tile, 4 waves of 128 x 128 accumulators each: a fragment read from LDS feeds twice as many matrix instructions,
//         which pays where nothing but the main loop counts (FP8, plain store, a tile for every CU)
using CfgQ256 = GemmCfg<256, 256, 2, 2, 128, 2, 1>;
//   N128, N256: attention's dV and dK (TN, up to 64 columns): 128 or 256 rows of the result by 64 columns, three or two
//         workgroups' worth of loads in flight per CU instead of a 128 x 128 tile whose right half is empty; two instructions of 32 x 32
//         results per k-step and wave (eight of 16 x 16: attention forward + backward of 1024 heads, us, 128 x 64 77.2 -> 77.6, 64 x 64 41.1 -> 41.4,
//         128 x 32 61.4 -> 61.9, 32 x 64 29.97 -> 30.4; 256 heads, 512 x 64 276.4 -> 276.9)
using CfgN128 = GemmCfg<128, 64, 4, 1, 128, 3, 2, 1, false>;
using CfgN256 = GemmCfg<256, 64, 8, 1, 128, 2, 1, 1, false>;

inline long ceil_div(long a, long b) { return (a + b - 1) / b; }

// All windows below are stated in units of the device's CU count (MI355X: 256), read from the device.
inline long cu_count() { return device_info().cus; }

// The large tile needs the output to cover the CUs about one and a half times, or at most once with three
// quarters of them busy (BERT-base on 256 CUs: 4096 x 3072 -> 192 tiles; backward of layer 2 there 67 -> 62 us); in
// between the small tile (two workgroups per CU, four times as many tiles) keeps more of the chip busy.
inline bool use_big_tile(long M, long N, int splits) {
  const long t = ceil_div(M, 256) * ceil_div(N, 256) * splits, cu = cu_count();
  return 2 * t >= 3 * cu || (4 * t >= 3 * cu && t <= cu);
}

// ... and for a single forward or grad_X product: more small tiles than fit two per CU, but large ones that fit one, instead of a
// second round of a few small tiles.  us, D128 -> D256: FP8 3136 x 2640, K = 4096 60.3 -> 40.6, FP16 11936 x 992, K = 3280 relu' 112 -> 88,
// 6000 x 1552, K = 1504 51.3 -> 35.1; over 160 drawn products of the window, plain and relu, the geometric mean is 0.87 from 768 to 2048 bytes
// of reduction (7 of 72 slower, by 2 to 8 %) and 0.74 beyond (none slower); below 768 bytes up to 9 % slower.  The arithmetic GELU and GELU', whose epilogue eight waves hardly
// speed up, need twice the reduction (short_gain; whether or not tables are ready: they still need a workspace and the copies they are
// made for).  D256 / D128 at 768 to 1024 / 1280 / 1536 bytes, geometric means over 210 drawn products: FP16 forward 1.04 / 1.00 / 0.99 (up to 1.16),
// GELU' 1.09 / 1.01 / 0.99 (up to 1.21), FP8 forward 0.99 / 0.95 / 0.91 (up to 1.17), which keeps 768 where the tables are ready (a test holds
// 3136 x 2640, K = 784 with an FP16 copy to D256).
inline bool use_big_single(const GemmProblem& p, bool short_gain) {
  if (use_big_tile(p.M, p.N, 1)) return true;
  const long t = ceil_div(p.M, 256) * ceil_div(p.N, 256), t128 = ceil_div(p.M, 128) * ceil_div(p.N, 128), cu = cu_count();
  return (p.a_kc || p.b_kc) && t128 > 2 * cu && t <= cu && p.K * (p.a_dt == US_F16 ? 2 : 1) >= (short_gain ? 1536 : 768);
}

// FP16 products whose output is covered exactly by 256 x 192 tiles, at most one per CU and at least seven eighths of
// the CUs busy
inline bool use_wide_tile(long M, long N) {
  const long t = ceil_div(M, 256) * ceil_div(N, 192), cu = cu_count();
  return N % 192 == 0 && t <= cu && 8 * t >= 7 * cu;
}

// grad_W whose 128 x 128 tiles just about cover the CUs once (C3: 4096 x 1024 -> 256 tiles): instead of
// cutting the long token reduction into slices that travel through HBM, two wave groups of one
// workgroup share it and add up in LDS.  A stage is at most 256 tokens long; a token count that
// is no multiple of it leaves part of the last stage empty, which pays as long as that is at most an eighth of the loop
// (2000 x 1552 x 2064 in FP8: layer 77.6 us with slices, 70.1 with the wave-split tile).
inline bool use_wave_split_tile(long M, long N, long K) {
  const long tiles = ceil_div(M, 128) * ceil_div(N, 128), cu = cu_count();
  return !use_big_tile(M, N, 1) && K >= 1024 && 8 * (ceil_div(K, 256) * 256 - K) <= K && 2 * tiles >= cu && tiles <= cu;
}

// The direct kernels address an operand with 32-bit offsets inside a tile of at most 256 rows (or 256 k-rows), and a result with
// 32-bit offsets inside 32 rows; longer row pitches (16 MB and more, 128 MB of an FP32 result) go to the register-staged kernel
// with its 64-bit addresses.
inline bool offsets_fit(const GemmProblem& p) {
  const long es = p.a_dt == US_F16 ? 2 : 1, ld = p.lda > p.ldb ? p.lda : p.ldb;
  return ld * es < (1l << 24) - 4096 && p.ldc < (1l << 25);
}

// Which tile of the few-tiles kernel (us_gemm_small.h) a product takes: the smallest of 32 x 32, 32 x 64 and 64 x 64 that
// gives every CU at most one tile; none if even 64 x 64 tiles outnumber the CUs.  Measured back to back, one box, us before
// (128 x 128 tiles; for 5 us the host's call rate is the limit) -> with these tiles, FP8 / FP16:
//   64 x 1024, K = 4096, forward   14.1 -> 6.1 / 28.0 -> 7.2   32 x 32     (32 x 64: 6.6 / 9.3)
//   512 x 1024, K = 1024, forward   7.8 -> 5.2 / 11.1 -> 5.7   32 x 64     (32 x 32: 6.1 / 7.2; 64 x 64: 5.6 / 6.6)
//   1024 x 1024, K = 4096, grad_X  14.9 -> 10.9 / 27.9 -> 19.1  64 x 64
//   64 x 16384, K = 4096, forward  16.8 -> 16.1 / 30.4 -> 25.6  64 x 64
//   1024 x 2048, K = 512, forward   5.4 -> 9.4 / 7.6 -> 10.1   64 x 64, two rounds: not taken
// grad_W, against 128 x 128 tiles with K slices: 1024 x 1024, K = 1024 11.7 -> 6.3 / 14.0 -> 6.6, 768 x 768, K = 4096
// 16.4 -> 10.2 / 20.4 -> 14.5, but 1024 x 1024, K = 16384 28.2 -> 43.1 / 53.1 -> 59.1.  From 4096 tokens on it keeps the slices:
// between 4096 and about 8192 it would still gain, but the tests hold 256 x 3072 over 4096 tokens to the slices.
enum class SmallTileChoice { None, T32x32, T32x64, T64x64 };     // in order of size
using CfgT32x32 = SmallCfg<1, 1, 2>;     // (a paired launch puts two workgroups on a CU, which leaves two stages per wave)
using CfgT32x64 = SmallCfg<1, 2, 3>;
using CfgT64x64 = SmallCfg<2, 2, 2>;
inline SmallTileChoice small_tile_choice(const GemmProblem& p) {
  const long cu = cu_count();
  if (p.batch > 1 || (!p.a_kc && !p.b_kc && p.K >= 4096)) return SmallTileChoice::None;
  const long t64 = ceil_div(p.M, 64) * ceil_div(p.N, 64);
  if (t64 > cu) return SmallTileChoice::None;
  // (the tests hold 4096 x 256 to the wave-split 128 x 128 tile)
  if (t64 == cu && p.M >= 16 * p.N) return SmallTileChoice::None;
  if (ceil_div(p.M, 32) * ceil_div(p.N, 32) <= cu) return SmallTileChoice::T32x32;
  return ceil_div(p.M, 32) * ceil_div(p.N, 64) <= cu ? SmallTileChoice::T32x64 : SmallTileChoice::T64x64;
}

// Forward and grad_X products whose 128 x 128 tiles give every CU at most one: the wave-split tile (W128), with its eight waves and
// four stages, where the reduction is long enough to fill them.  us, D128 -> W128:
//   plain store  FP8 2048 x 2048, K = 1024 7.6 -> 8.7, K = 4096 24.1 -> 20.3, 1024 x 1536, K = 3072 14.0 -> 12.5 (from K = 1536 on);
//                FP16 2048 x 2048, K = 512 8.1 -> 9.2, K = 1024 12.2 -> 12.9, K = 4096 50.0 -> 38.2, 4096 x 1024, K = 2048 25.4 -> 22.4
//   activation and its derivative, whose epilogue eight waves halve: FP8 2048 x 2048, K = 512 gelu 9.7 -> 10.0, relu 10.1 -> 9.4,
//                K = 1024 11.5 -> 11.3 and 12.0 -> 10.8, relu' 13.4 -> 11.9; FP16 K = 512 11.8 -> 11.6, 12.1 -> 11.0, 13.5 -> 11.9,
//                K = 4096 52 -> 40, 51 -> 42 (from 1024 bytes of K on)
inline bool use_wave_split_small(const GemmProblem& p, int epi) {
  if (ceil_div(p.M, 128) * ceil_div(p.N, 128) > cu_count()) return false;
  const long kb = p.K * (p.a_dt == US_F16 ? 2 : 1);
  if (epi == EPI_GELU || epi == EPI_GELU_GRAD) return kb >= 1024;
  return kb >= (epi == EPI_STORE ? 1536 : 1024) && p.K >= 1024;
}

inline GemmArgs make_args(const GemmProblem& p, long k_per_split, int BM, int BN) {
  GemmArgs g{};
  g.A = (const uint8_t*)p.A;
  g.B = (const uint8_t*)p.B;
  g.C = p.C;
  g.M = p.M; g.N = p.N; g.K = p.K;
  g.lda = p.lda; g.ldb = p.ldb; g.ldc = p.ldc;
  g.k_per_split = k_per_split;
  g.scale = p.scale;
  g.epi_scale = p.epi_scale;
  g.skip_scale = p.skip_scale;
  g.act = p.act;
  g.Zpre = (const _Float16*)p.Zpre;
  g.aux16 = (_Float16*)p.aux16;
  g.aux8 = (uint8_t*)p.aux8;
  g.partial = (float*)p.workspace;
  g.table = (const uint8_t*)p.table;
  g.bias = (const _Float16*)p.bias;
  g.colsum = (float*)p.colsum;
  if (p.batch > 1) {
    const long es = (p.a_dt == US_F16) ? 2 : 1;
    g.batch_a = p.batch_a * es;
    g.batch_b = p.batch_b * es;
    g.batch_c = p.batch_c * (p.c_dt == US_F32 ? 4 : 2);
  }
  const long tiles_m = ceil_div(p.M, BM), tiles_n = ceil_div(p.N, BN);
  const int nxcd = device_info().xcds;
  int gm, gn;
  choose_xcd_grid(tiles_m, tiles_n, nxcd, BM, BN, gm, gn);
  // bands 8 tiles wide: the 32 (one per CU) or 64 (two per CU) tiles that run together on an XCD form 4 x 8 or 8 x 8.
  // (Measured for the large tile: 4 wide was 3 us slower on the 8192 x 4096 x 1024 product with the GELU epilogue,
  // 16 and 32 equal to 8; the other tile shapes show no difference between 2 and 16.)
  g.walk = TileWalk(tiles_m, tiles_n, nxcd, gm, gn, 8);
  return g;
}

// Bytes of reduction up to which a tile takes the matrix instructions of 32 x 32 results (a second copy of its kernel, Short<Cfg>): no more stages than the
// ring has slots, on 128 x 128 FP16 tiles of grad_W one more.  Power, which the 16 x 16 forms are for, does not limit such a product, and twice as
// many or twice as large fragments per k-step hold up its start.  us, 16 x 16 -> 32 x 32 form:
//   128 x 128 FP16, K = 128: 8192 x 512 NN 4.58 -> 4.48, 3072 x 1024 NT 4.22 -> 4.05, 2048 x 2560 TN 5.13 -> 4.98; K = 192: TN 5.79 -> 5.66, 3072 x 1024 NT even,
//     2048 x 3072 NN 5.70 -> 5.73; from 256 on the 16 x 16 form by 0 to 7 %.  256 x 192, 4096 x 3072, K = 64 7.81 -> 7.71, K = 128 8.95 -> 8.88, K = 192 9.90 -> 9.96
//   256 x 256 FP8, K = 128: 8192 x 4096 NN 15.97 -> 15.84, 4096 x 3072 NN 7.48 -> 7.46, 11008 x 4096 TN 21.8 -> 21.6; K = 256: 18.3 -> 18.3, 25.6 -> 25.3; K = 320 even or
//     slower.  grad_X (NT) is even at K = 16 and faster with 16 x 16 from 64 on, and so is the 256 x 256 FP16 tile
//   layers forward and backward: FP16 192 x 3072 x 1536 24.8 -> 24.5, 128 x 2048 x 3072 21.9 -> 21.8; none of 177 products and passes slower by more than 0.8 %, which is their spread
template <class Cfg>
using Short = GemmCfg<Cfg::BM, Cfg::BN, Cfg::WAVES_M, Cfg::WAVES_N, Cfg::BKB, Cfg::NST, Cfg::MINB, Cfg::WAVES_K, false>;
template <class Cfg, bool FP8, bool A_KC, bool B_KC>
constexpr long short_reduction() {
  if (FP8) return std::is_same<Cfg, CfgD256>::value && !(A_KC && B_KC) ? Cfg::NST * Cfg::BKB : 0;
  if (std::is_same<Cfg, CfgE192>::value) return Cfg::NST * Cfg::BKB;
  if (std::is_same<Cfg, CfgD128>::value) return (A_KC || B_KC ? Cfg::NST : Cfg::NST + 1) * Cfg::BKB;
  return 0;
}

template <bool DIRECT, class Cfg, bool FP8, int FA, int FB, bool A_KC, bool B_KC, int EPI, bool WIDE>
hipError_t launch_one(const GemmProblem& p, int splits, long k_per_split, hipStream_t st) {
  constexpr long SHORT = DIRECT ? short_reduction<Cfg, FP8, A_KC, B_KC>() : 0;
  if constexpr (SHORT > 0) {
    if (k_per_split * (FP8 ? 1 : 2) <= SHORT) return launch_one<DIRECT, Short<Cfg>, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, splits, k_per_split, st);
  }
  using Tile = typename std::conditional<DIRECT, DirectTile<Cfg, FP8, A_KC, B_KC, WIDE, EPI>,
                                         StagedTile<Cfg, FP8, A_KC, B_KC, WIDE, EPI>>::type;
  constexpr int LDS = Tile::LDS_BYTES;
  void (*kern)(GemmArgs);
  if constexpr (DIRECT) kern = gemm_direct_kernel<Cfg, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>;
  else kern = gemm_staged_kernel<Cfg, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>;
  note_gemm_launch(DIRECT ? "direct" : "staged", Cfg::BM, Cfg::BN, Cfg::WAVES_K, Cfg::NST, FP8, A_KC, B_KC, EPI, WIDE, splits,
                   std::is_same<Cfg, CfgQ256>::value ? Cfg::WAVES : 0);
  static FuncConfig cfg;           // raising the dynamic-LDS limit: once per function and device
  if (hipError_t e = cfg.ensure((const void*)kern, LDS); e != hipSuccess) return e;
  const GemmArgs g = make_args(p, k_per_split, Cfg::BM, Cfg::BN);
  const long tiles = ceil_div(p.M, Cfg::BM) * ceil_div(p.N, Cfg::BN);
  dim3 grid((unsigned)tiles, (unsigned)splits, (unsigned)(p.batch > 1 ? p.batch : 1));
  kern<<<grid, Cfg::THREADS, LDS, st>>>(g);
  return hipGetLastError();
}

template <class Cfg, bool FP8, int FA, int FB, bool A_KC, bool B_KC, int EPI, bool WIDE>
hipError_t launch_small(const GemmProblem& p, hipStream_t st) {
  constexpr int LDS = SmallTile<Cfg, FP8, A_KC, B_KC>::LDS_BYTES;
  auto kern = gemm_small_kernel<Cfg, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>;
  note_gemm_launch("direct", Cfg::BM, Cfg::BN, Cfg::WAVES, Cfg::NST, FP8, A_KC, B_KC, EPI, WIDE, 1);
  static FuncConfig cfg;
  if (hipError_t e = cfg.ensure((const void*)kern, LDS); e != hipSuccess) return e;
  const GemmArgs g = make_args(p, p.K, Cfg::BM, Cfg::BN);
  kern<<<(unsigned)(ceil_div(p.M, Cfg::BM) * ceil_div(p.N, Cfg::BN)), Cfg::THREADS, LDS, st>>>(g);
  return hipGetLastError();
}

template <bool FP8, int FA, int FB, bool A_KC, bool B_KC, int EPI, bool WIDE>
hipError_t launch_sized(const GemmProblem& p, int splits, long k_per_split, hipStream_t st) {
  // (K slices are for outputs of few tiles; an operand pitch of 16 MB makes tens of thousands)
  if constexpr (EPI == EPI_PARTIAL) {
    if (!offsets_fit(p)) return hipErrorInvalidValue;
  } else {
    if (!offsets_fit(p)) return launch_one<false, CfgS128, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, splits, k_per_split, st);
    const SmallTileChoice c = small_tile_choice(p);
    if (c == SmallTileChoice::T32x32) return launch_small<CfgT32x32, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, st);
    if (c == SmallTileChoice::T32x64) return launch_small<CfgT32x64, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, st);
    if (c == SmallTileChoice::T64x64) return launch_small<CfgT64x64, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, st);
  }
  const bool batched = p.batch > 1;      // the tile count that decides is the whole batch's
  if constexpr (!FP8 && (A_KC || B_KC) && EPI == EPI_STORE && !WIDE) {
    if (splits == 1 && !batched && use_wide_tile(p.M, p.N))
      return launch_one<true, CfgE192, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, splits, k_per_split, st);
  }
  if constexpr (FP8 && EPI == EPI_STORE && !WIDE) {
    // a large tile for every CU and a long reduction: the wave's larger tile (LDS reads 64 instead of 96 bytes per clock and CU next to the
    // matrix core) beats the second wave per SIMD, by the more the fuller the last round.  us, D256 -> Q256 (tiles per CU), one process, in turn:
    //   NN  4096 x 4096, K = 4096 (1) 48.5 -> 47.9, 4096 x 8192, K = 5120 (2) 116.2 -> 115.8, 6992 x 6992, K = 4096 (3.1) 179 -> 173, 16384 x 4096 (4) 192 -> 191,
    //       7168 x 4096 (1.75) even; worst, a last round up to half full: 6144 x 4096 (1.5) 82.1 -> 83.0, 5104 x 5136 (1.6) 103.4 -> 104.5, 9216 x 4096 (2.25) 125.4 ->
    //       126.4; shorter ones, older figures: 6144 x 4096, K = 2560 (1.5) 58.6 -> 59.9, K = 3072 67.5 -> 68.5, but 8192 x 4096, K = 3072 (2) 78.1 -> 76.1
    //   NT  8192 x 4096, K = 2048 (2) 52.9 -> 52.5, 10240 x 5120, K = 3072 (3.1) 133.6 -> 131.6, 6144 x 6144, K = 4096 (2.25) 124.6 -> 122.9; worst 5104 x 5136,
    //       K = 2064 (1.6) 61.0 -> 61.9;  8192 x 4096, K = 1024 no difference
    //   TN  4096 x 4096, K = 4096 (1) 48.9 -> 48.1, 7168 x 4096 (1.75) 90.0 -> 88.6, 12288 x 4096 (3) 147.9 -> 144.2, 6144 x 6144, K = 8192 (2.25) 239 -> 235; worst
    //       5104 x 5136, K = 4144 (1.6) 98.2 -> 100.0, K = 8192 181 -> 183, 6000 x 6000, K = 4096 (2.25) 136.3 -> 138.6
    // (53 products: geometric mean 0.9985)
    // FP16 868 -> 884 and more: not taken
    if (!batched && splits == 1 && use_big_tile(p.M, p.N, 1) && ceil_div(p.M, 256) * ceil_div(p.N, 256) >= cu_count() && p.K >= (A_KC && B_KC ? 2048 : 4096))
      return launch_one<true, CfgQ256, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, splits, k_per_split, st);
  }
  if constexpr ((A_KC || B_KC) && !WIDE) {
    const bool short_gain = p.act == 0 && (EPI == EPI_GELU_GRAD || (EPI == EPI_GELU && !(FP8 && p.tables_ready)));
    if (!batched && splits == 1 && use_big_single(p, short_gain))
      return launch_one<true, CfgD256, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, splits, k_per_split, st);
  }
  if (use_big_tile(p.M, p.N, splits * (int)(batched ? p.batch : 1)) && (!batched || (p.M >= 256 && p.N >= 256)))
    return launch_one<true, CfgD256, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, splits, k_per_split, st);
  if (batched) return launch_one<true, CfgD128, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, splits, k_per_split, st);
  if constexpr (FP8 && (A_KC || B_KC) && (EPI == EPI_STORE || EPI == EPI_RESIDUAL) && !WIDE) {
    // an output of about one tile of 256 x 128 per CU (BERT-large: Linear 2, 8192 x 1024 -> 256): two wave groups
    // (40 against 43 us forward, 35 against 37 us in the grad_X layout; FP8 only, not measured for FP16)
    const long t_mid = ceil_div(p.M, 256) * ceil_div(p.N, 128);
    if (splits == 1 && 4 * t_mid >= 3 * cu_count() && t_mid <= cu_count() && p.K >= 1024)
      return launch_one<true, CfgM256, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, splits, k_per_split, st);
  }
  if constexpr ((A_KC || B_KC) && (EPI == EPI_STORE || EPI == EPI_RESIDUAL || EPI == EPI_GELU || EPI == EPI_GELU_GRAD) && !WIDE) {
    if (splits == 1 && use_wave_split_small(p, EPI)) return launch_one<true, CfgW128, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, splits, k_per_split, st);
  }
  if constexpr (FP8 && A_KC && !B_KC && !WIDE) {
    // FP8 forward with a few tiles more than CUs: 128 x 256 tiles, one per CU, instead of a CU here and there with two small ones
    // that the others wait for.  It pays with a short reduction, or with two or four columns of tiles, and not where the last row of
    // tiles is mostly empty: then the second small tiles cost little.  us back to back on the same operands, D128 -> H256, plain /
    // relu / gelu:
    //   2000 x 2064, K = 1552 13.8 -> 12.7, 18.2 -> 16.8, 20.8 -> 18.2;  K = 4096 29.0 -> 32.3, 33.7 -> 36.5, 36.5 -> 37.8
    //   2176 x 2048, K = 1552 12.7 -> 12.0, 17.2 -> 16.5, 18.0 -> 17.9;  K = 2048 15.4 -> 17.3, 20.0 -> 22.1, 21.2 -> 23.4
    //   4224 x 1024, K = 1024 10.9 -> 9.4, 15.4 -> 13.8, 16.4 -> 15.0;  K = 6144 50.3 -> 44.3, 55.1 -> 48.8, 56.2 -> 50.2
    //   8320 x 512, K = 2048 17.7 -> 16.7, 22.2 -> 21.4, 23.3 -> 22.7;  5632 x 768, K = 2048 16 to 19 % slower
    //   2080 x 2048, K = 1024 9.7 -> 9.7, 12.5 -> 14.3, 12.6 -> 15.4;  4112 x 1024, K = 2048 2 % faster, 3 and 12 % slower
    // (grad_X with relu' 22.8 -> 23.5 and FP16 25.5 -> 27.8: not taken; 3072 x 2048, 384 tiles, no difference; the tests hold 288
    // to the small tile)
    const long t = ceil_div(p.M, 128) * ceil_div(p.N, 128), cu = cu_count();
    const bool short_k = p.K >= 1024 && p.K < 1664, even_columns = p.K >= 1024 && p.N <= 1024 && p.N % 512 == 0;
    if (t > cu && 8 * t < 9 * cu && ceil_div(p.M, 128) * ceil_div(p.N, 256) <= cu && (p.M - 1) % 128 >= 63 && (short_k || even_columns))
      return launch_one<true, CfgH256, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, splits, k_per_split, st);
  }
  if constexpr (!A_KC && !B_KC && EPI == EPI_STORE) {
    if (splits == 1 && use_wave_split_tile(p.M, p.N, p.K))
      return launch_one<true, CfgK128, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, splits, k_per_split, st);
  }
  return launch_one<true, CfgD128, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(p, splits, k_per_split, st);
}

// The table-driven GELU epilogues exist for the large tile of the direct kernel only (the table needs 64-73 KB of LDS next to the
// strips).  Where the large tile pays for a single product only, it does not pay for building the table as well (4 us).
inline bool table_path_ok(const GemmProblem& p) {
  return p.table != nullptr && p.act == 0 && offsets_fit(p) && (use_big_tile(p.M, p.N, 1) || (p.tables_ready && use_big_single(p, false)));   // the tables are gelu's
}

// ... and for the 256 x 192 tile (FP16, no column sums: a lane of its epilogue does not keep to the same columns)
inline bool wide_table_path_ok(const GemmProblem& p) {
  return p.table != nullptr && p.act == 0 && offsets_fit(p) && p.colsum == nullptr && use_wide_tile(p.M, p.N);
}

template <class Cfg>
hipError_t launch_two_batches(const GemmProblem& p, const GemmProblem& q, hipStream_t st) {
  constexpr int LDS = DirectTile<Cfg, false, false, false, false>::LDS_BYTES;
  auto kern = gemm_two_batches_kernel<Cfg, false, 0, 0, false, false>;
  for (int i = 0; i < 2; ++i) note_gemm_launch("pair", Cfg::BM, Cfg::BN, 1, Cfg::NST, false, false, false, EPI_STORE, false, 1);
  static FuncConfig cfg;
  if (hipError_t e = cfg.ensure((const void*)kern, LDS); e != hipSuccess) return e;
  GemmArgs a = make_args(p, p.K, Cfg::BM, Cfg::BN), b = make_args(q, q.K, Cfg::BM, Cfg::BN);
  a.batch_a = p.batch_a * 2; a.batch_b = p.batch_b * 2; a.batch_c = p.batch_c * 2;      // (also for a batch of one)
  b.batch_a = q.batch_a * 2; b.batch_b = q.batch_b * 2; b.batch_c = q.batch_c * 2;
  const long tiles_m = ceil_div(p.M, Cfg::BM), tiles_n = ceil_div(p.N, Cfg::BN), tiles = tiles_m * tiles_n;
  const int nxcd = device_info().xcds;
  a.walk = b.walk = TileWalk(tiles_m, tiles_n, nxcd, 0, 0, 8);       // the tiles of an item stay together
  BatchWalk w;
  w.by_xcds = FastDiv::by((uint32_t)nxcd);
  w.by_tiles = FastDiv::by((uint32_t)tiles);
  w.xcds = (uint32_t)nxcd;
  w.tiles = (uint32_t)tiles;
  w.batch = (int)p.batch;
  kern<<<(unsigned)(tiles * ceil_div(2 * p.batch, nxcd) * nxcd), Cfg::THREADS, LDS, st>>>(w, a, b);
  return hipGetLastError();
}

// Plain store epilogue: FP16 or FP32 output.
template <bool FP8, int FA, int FB, bool A_KC, bool B_KC>
hipError_t launch_store(const GemmProblem& p, hipStream_t st) {
  if (p.c_dt == US_F32) return launch_sized<FP8, FA, FB, A_KC, B_KC, EPI_STORE, true>(p, 1, p.K, st);
  return launch_sized<FP8, FA, FB, A_KC, B_KC, EPI_STORE, false>(p, 1, p.K, st);
}

hipError_t launch_splitk_reduce(const float* partial, void* out, long total, int splits, float scale, bool out_is_f32,
                                hipStream_t st);

// Families (defined one per translation unit).
hipError_t gemm_nn_f16(const GemmProblem& p, hipStream_t st);   // forward:  A K-contig, B K-strided
hipError_t gemm_nn_fp8(const GemmProblem& p, hipStream_t st);
hipError_t gemm_nt_f16(const GemmProblem& p, hipStream_t st);   // grad_X:   both K-contig
hipError_t gemm_nt_fp8(const GemmProblem& p, hipStream_t st);
hipError_t gemm_tn_f16(const GemmProblem& p, hipStream_t st);   // grad_W:   both K-strided, split-K
hipError_t gemm_tn_fp8(const GemmProblem& p, hipStream_t st);

}  // namespace us
