// Both products of a layer's backward pass (grad_X and grad_W) in one launch, for the combinations of tile shapes listed
// below: see gemm_pair_kernel.
#include "us_gemm_dispatch.h"

namespace us {

namespace {

template <class KA, class KB>
hipError_t launch_pair(const GemmProblem& dx, const GemmProblem& dw, hipStream_t st) {
  constexpr int LDS = KA::Tile::LDS_BYTES > KB::Tile::LDS_BYTES ? KA::Tile::LDS_BYTES : KB::Tile::LDS_BYTES;
  note_gemm_launch("pair", KA::BM, KA::BN, KA::WAVES_K, KA::NST, KA::IS_FP8, KA::A_KC_, KA::B_KC_, KA::EPI_, false, 1);
  note_gemm_launch("pair", KB::BM, KB::BN, KB::WAVES_K, KB::NST, KB::IS_FP8, KB::A_KC_, KB::B_KC_, KB::EPI_, false, 1);
  static FuncConfig cfg;
  if (hipError_t e = cfg.ensure((const void*)gemm_pair_kernel<KA, KB>, LDS); e != hipSuccess) return e;
  const GemmArgs a = make_args(dx, dx.K, KA::BM, KA::BN);
  const GemmArgs b = make_args(dw, dw.K, KB::BM, KB::BN);
  const long tiles_a = ceil_div(dx.M, KA::BM) * ceil_div(dx.N, KA::BN), tiles_b = ceil_div(dw.M, KB::BM) * ceil_div(dw.N, KB::BN);
  gemm_pair_kernel<KA, KB><<<(unsigned)(tiles_a + tiles_b), KA::THREADS, LDS, st>>>((int)tiles_b, a, b);
  return hipGetLastError();
}

// grad_W in a pair on 256 x 128 tiles that take about half of the CUs (BERT-large: 4096 x 1024 -> 128 tiles).  Such a
// tile needs 36 % less CU time than two wave-split 128 x 128 tiles, but covers only half of the chip and runs twice as
// long: on its own that is slower, in a pair the grad_X tiles take the other CUs from the start and the launch ends
// when it would have ended with grad_W spread over all CUs, minus the CU time saved.  With fewer than 112 tiles the
// long tiles outlast the rest of the launch (BERT-base, 72 tiles: measured slower).
bool long_tile_ok(const GemmProblem& dw) {
  const long t = ceil_div(dw.M, 256) * ceil_div(dw.N, 128), cu = cu_count();
  return 16 * t >= 7 * cu && 2 * t <= cu && t % device_info().xcds == 0;
}

// grad_X without an activation derivative whose 256 x 256 tiles, together with grad_W's long tiles, give every CU one
// tile of about the same length (BERT-large layer 1: 128 + 128)
bool one_round_ok(const GemmProblem& dx, const GemmProblem& dw) {
  const long t = ceil_div(dx.M, 256) * ceil_div(dx.N, 256) + ceil_div(dw.M, 256) * ceil_div(dw.N, 128);
  return long_tile_ok(dw) && (dx.epi == US_EPI_NONE || dx.epi == US_EPI_RESIDUAL) && 8 * t >= 7 * cu_count() && t <= cu_count() &&
         dx.K >= 2048;
}

// grad_X on so few 128 x 128 tiles that the CUs get at most one each (wave-split small tile)
bool small_tile_ok(const GemmProblem& dx) {
  const long t = ceil_div(dx.M, 128) * ceil_div(dx.N, 128);
  return t <= cu_count() && dx.K >= 1024 && !use_big_tile(dx.M, dx.N, 1);
}

// grad_X without an epilogue whose 256 x 128 tiles cover the CUs about once
bool mid_tile_ok(const GemmProblem& dx) {
  const long t = ceil_div(dx.M, 256) * ceil_div(dx.N, 128);
  return (dx.epi == US_EPI_NONE || dx.epi == US_EPI_RESIDUAL) && 4 * t >= 3 * cu_count() && 4 * t <= 5 * cu_count();
}

// grad_X without an epilogue whose 256 x 128 tiles, together with grad_W's tiles, give every CU at most one tile
// (BERT-base layer 1: 96 + 144): one round instead of 192 + 144 small tiles in one and a third
bool mid_one_round_ok(const GemmProblem& dx, const GemmProblem& dw) {
  const long tw = long_tile_ok(dw) ? ceil_div(dw.M, 256) * ceil_div(dw.N, 128) : ceil_div(dw.M, 128) * ceil_div(dw.N, 128);
  const long t = ceil_div(dx.M, 256) * ceil_div(dx.N, 128) + tw;
  return (dx.epi == US_EPI_NONE || dx.epi == US_EPI_RESIDUAL) && t <= cu_count() && 8 * t >= 7 * cu_count() && dx.K >= 2048;
}

// grad_X with the table-driven GELU' whose large tiles fit one round on their own but not next to grad_W's tiles
// (BERT-base layer 2: 192 + 144 on 256 CUs): twice as many tiles of 128 x 256 fill the second round's gaps
// (FP16: 62.7 -> 59.5 us; FP8 operands at the same shape: 46.6 -> 43.1 us; same box each)
bool half_tile_ok(const GemmProblem& dx, const GemmProblem& dw) {
  const long tw = long_tile_ok(dw) ? ceil_div(dw.M, 256) * ceil_div(dw.N, 128) : ceil_div(dw.M, 128) * ceil_div(dw.N, 128);
  const long t = ceil_div(dx.M, 256) * ceil_div(dx.N, 256);
  return t <= cu_count() && t + tw > cu_count();
}

template <bool FP8, class KW>
hipError_t launch_pair_kw(const GemmProblem& dx, const GemmProblem& dw, hipStream_t st) {
  constexpr int FG = FP8 ? 1 : 0;                     // gradient operand format (E5M2) where it applies
  if (dx.epi == US_EPI_GELU_GRAD && small_tile_ok(dx))
    return launch_pair<GemmKind<CfgW128, FP8, FG, 0, true, true, EPI_GELU_GRAD, false>, KW>(dx, dw, st);
  if (dx.epi == US_EPI_GELU_GRAD && !use_big_tile(dx.M, dx.N, 1))
    return launch_pair<GemmKind<CfgM256, FP8, FG, 0, true, true, EPI_GELU_GRAD, false>, KW>(dx, dw, st);
  if (dx.epi == US_EPI_GELU_GRAD) {
    GemmProblem q = dx;
    q.table = (char*)dx.table + kGeluSlopeTableOffset;
    if (!dx.tables_ready) {
      hipError_t e = launch_gelu_slope_table(q.table, dx.epi_scale, st);
      if (e != hipSuccess) return e;
    }
    if (half_tile_ok(dx, dw))
      return launch_pair<GemmKind<CfgH256, FP8, FG, 0, true, true, EPI_GELU_GRAD_TAB, false>, KW>(q, dw, st);
    return launch_pair<GemmKind<CfgD256, FP8, FG, 0, true, true, EPI_GELU_GRAD_TAB, false>, KW>(q, dw, st);
  }
  // the large tile also when it and grad_W's long tiles fill the CUs exactly once
  const bool big = use_big_tile(dx.M, dx.N, 1) || (KW::BM == 256 && one_round_ok(dx, dw));
  if (dx.epi == US_EPI_RESIDUAL) {
    if (big) return launch_pair<GemmKind<CfgD256, FP8, FG, 0, true, true, EPI_RESIDUAL, false>, KW>(dx, dw, st);
    if (small_tile_ok(dx) && !mid_tile_ok(dx) && !mid_one_round_ok(dx, dw))
      return launch_pair<GemmKind<CfgW128, FP8, FG, 0, true, true, EPI_RESIDUAL, false>, KW>(dx, dw, st);
    return launch_pair<GemmKind<CfgM256, FP8, FG, 0, true, true, EPI_RESIDUAL, false>, KW>(dx, dw, st);
  }
  if (big) return launch_pair<GemmKind<CfgD256, FP8, FG, 0, true, true, EPI_STORE, false>, KW>(dx, dw, st);
  if (mid_one_round_ok(dx, dw))
    return launch_pair<GemmKind<CfgM256, FP8, FG, 0, true, true, EPI_STORE, false>, KW>(dx, dw, st);
  if (small_tile_ok(dx)) return launch_pair<GemmKind<CfgW128, FP8, FG, 0, true, true, EPI_STORE, false>, KW>(dx, dw, st);
  return launch_pair<GemmKind<CfgM256, FP8, FG, 0, true, true, EPI_STORE, false>, KW>(dx, dw, st);
}

template <bool FP8>
hipError_t launch_pair_typed(const GemmProblem& dx, const GemmProblem& dw, hipStream_t st) {
  constexpr int FG = FP8 ? 1 : 0;
  if (long_tile_ok(dw)) return launch_pair_kw<FP8, GemmKind<CfgM256, FP8, 0, FG, false, false, EPI_STORE, false>>(dx, dw, st);
  return launch_pair_kw<FP8, GemmKind<CfgK128, FP8, 0, FG, false, false, EPI_STORE, false>>(dx, dw, st);
}


// Both products on the few-tiles kernel, with the larger of the two tiles they would take alone: one launch instead of two
// of about 5 us each, most of which is the launch itself (FP16 layer of 256 x 256 x 1024, forward + backward: 17.8 -> 13.5 us).
bool small_pair_ok(const GemmProblem& dx, const GemmProblem& dw) {
  return small_tile_choice(dx) != SmallTileChoice::None && small_tile_choice(dw) != SmallTileChoice::None && offsets_fit(dx) &&
         offsets_fit(dw);
}

// Whether grad_W is written over something that grad_X reads or writes, or grad_X over what grad_W reads: such products need
// two launches, grad_X first.
bool halves_share_memory(const GemmProblem& dx, const GemmProblem& dw) {
  const size_t es = dx.b_dt == US_F16 ? 2 : 1, nw = (size_t)dw.M * dw.N, nx = (size_t)dx.M * dx.N;
  return overlap(dw.C, nw * 2, dx.B, nw * es) || overlap(dw.C, nw * 2, dx.Zpre, nx * 2) || overlap(dw.C, nw * 2, dx.C, nx * 2) ||
         overlap(dw.C, nw * 2, dx.aux8, nx) || overlap(dx.C, nx * 2, dw.A, nx * es) || overlap(dx.aux8, nx, dw.A, nx * es);
}

template <class Cfg, bool FP8, int EPI>
hipError_t launch_small_pair(const GemmProblem& dx, const GemmProblem& dw, hipStream_t st) {
  constexpr int LDX = SmallTile<Cfg, FP8, true, true>::LDS_BYTES, LDW = SmallTile<Cfg, FP8, false, false>::LDS_BYTES;
  constexpr int LDS = LDX > LDW ? LDX : LDW;
  note_gemm_launch("pair", Cfg::BM, Cfg::BN, Cfg::WAVES, Cfg::NST, FP8, true, true, EPI, false, 1);
  note_gemm_launch("pair", Cfg::BM, Cfg::BN, Cfg::WAVES, Cfg::NST, FP8, false, false, EPI_STORE, false, 1);
  static FuncConfig cfg;
  if (hipError_t e = cfg.ensure((const void*)gemm_small_pair_kernel<Cfg, FP8, EPI>, LDS); e != hipSuccess) return e;
  const GemmArgs a = make_args(dx, dx.K, Cfg::BM, Cfg::BN), b = make_args(dw, dw.K, Cfg::BM, Cfg::BN);
  const long ta = ceil_div(dx.M, Cfg::BM) * ceil_div(dx.N, Cfg::BN), tb = ceil_div(dw.M, Cfg::BM) * ceil_div(dw.N, Cfg::BN);
  gemm_small_pair_kernel<Cfg, FP8, EPI><<<(unsigned)(ta + tb), Cfg::THREADS, LDS, st>>>((int)tb, a, b);
  return hipGetLastError();
}

template <bool FP8, int EPI>
hipError_t launch_small_pair_sized(const GemmProblem& dx, const GemmProblem& dw, hipStream_t st) {
  const SmallTileChoice x = small_tile_choice(dx), w = small_tile_choice(dw), c = x > w ? x : w;
  if (c == SmallTileChoice::T32x32) return launch_small_pair<CfgT32x32, FP8, EPI>(dx, dw, st);
  if (c == SmallTileChoice::T32x64) return launch_small_pair<CfgT32x64, FP8, EPI>(dx, dw, st);
  return launch_small_pair<CfgT64x64, FP8, EPI>(dx, dw, st);
}

template <bool FP8>
hipError_t launch_small_pair_typed(const GemmProblem& dx, const GemmProblem& dw, hipStream_t st) {
  if (dx.epi == US_EPI_GELU_GRAD) return launch_small_pair_sized<FP8, EPI_GELU_GRAD>(dx, dw, st);
  if (dx.epi == US_EPI_RESIDUAL) return launch_small_pair_sized<FP8, EPI_RESIDUAL>(dx, dw, st);
  return launch_small_pair_sized<FP8, EPI_STORE>(dx, dw, st);
}

// Both products on eight-wave tiles, one per CU (launch_pair_typed chooses them).
bool eight_wave_pair_ok(const GemmProblem& dx, const GemmProblem& dw) {
  const bool big = use_big_tile(dx.M, dx.N, 1);
  const long t_mid = ceil_div(dx.M, 256) * ceil_div(dx.N, 128);
  // grad_X with the arithmetic activation-derivative epilogue on 256 x 128 tiles (an output too small for the large tile)
  const bool mid_act = dx.epi == US_EPI_GELU_GRAD && !big && 4 * t_mid >= 3 * cu_count() && t_mid <= 2 * cu_count();
  const bool small_pair = (small_tile_ok(dx) && !mid_tile_ok(dx)) || mid_act;
  if (!offsets_fit(dx) || !offsets_fit(dw) || !(big || mid_tile_ok(dx) || small_pair || one_round_ok(dx, dw) || mid_one_round_ok(dx, dw))) return false;
  if (dx.epi == US_EPI_GELU_GRAD && big && (!dx.table || dx.act != 0)) return false;   // large tile: table-driven epilogue only
  return use_wave_split_tile(dw.M, dw.N, dw.K);
}

// Both products on the four-wave 128 x 128 tile, two workgroups per CU, where all tiles of both are resident at once: on eight-wave
// tiles, one per CU, they take two rounds, the second half empty, or go out as two launches.  Two workgroups on a CU also fill
// each other's waits, and one's epilogue runs under the other's products.  us, without this rule -> with it, grad_X with relu' / plain:
//   2000 x 1552 x 2064 (208 + 221 tiles), relu' only, FP8 30.1 -> 22.7, FP16 46.4 -> 38.1
//   2048 x 2048 x 1536 (256 + 192) FP8 21.2 -> 15.2 / 19.2 -> 13.7;  3072 x 1536 x 1536 (288 + 144, two launches before) 30.9 -> 20.1 / 27.7 -> 19.1
//   2688 x 768 x 2304 (126 + 108, K slices before) 30.0 -> 18.0 / 28.4 -> 16.9;  640 x 3328 x 512 (130 + 104) 11.8 -> 7.0 / 9.8 -> 5.5
// over 200 drawn layers that this rule or the next one moves the geometric mean is 0.75, none slower by 1 %.  Not taken where one product's few tiles with a long reduction
// outlast the rest (3536 x 1056 x 976, 252 + 72: FP16 41.9 -> 48.1; 1792 x 1024 x 5632, 112 + 352: 35.7 -> 36.4), and where the
// eight-wave tiles fit one round (2320 x 816 x 3536 on 133 + 98: 25.6 -> 32.4; 3088 x 720 x 3280 FP16 53.4 -> 54.4).
bool all_resident_ok(const GemmProblem& dx, const GemmProblem& dw, long tx, long tw) {
  const long cu = cu_count();
  if (tx + tw > 2 * cu || 8 * tx < 3 * cu || 8 * tw < 3 * cu) return false;
  const long longer = dx.K > dw.K ? dx.K : dw.K, shorter = dx.K > dw.K ? dw.K : dx.K;
  if ((2 * tx < cu || 2 * tw < cu) && 2 * longer > 3 * shorter) return false;
  if (eight_wave_pair_ok(dx, dw)) {
    if (tx + tw <= cu) return false;
    const bool mid = mid_one_round_ok(dx, dw) || !small_tile_ok(dx);
    const long bx = mid ? ceil_div(dx.M, 256) * ceil_div(dx.N, 128) : tx, bw = long_tile_ok(dw) ? ceil_div(dw.M, 256) * ceil_div(dw.N, 128) : tw;
    if (bx + bw <= cu) return false;
    // (a plain grad_X next to fewer tiles would gain as well, 2048 x 1536 x 2048 FP8 21.8 -> 15.3, 2000 x 1552 x 2064 29.7 -> 22.3, but the
    // tests hold 2000 x 1552 x 2064 and 1024 x 2048 x 1536 to the eight-wave tiles)
    if (dx.epi == US_EPI_NONE && 4 * (tx + tw) < 7 * cu) return false;
  }
  return true;
}

// The same tiles where all_resident_ok does not hold: more of them than slots, or one product's few tiles next to many.  The launch
// then lasts as long as its slots are evenly filled, so its longest tile is held against the work of one CU (both in bytes of
// reduction; a tile's prologue and epilogue take as long as about 1000 more).  us, two launches -> this:
//   a derivative up to 7/8 of the slots:  GELU' 1568 x 2624 x 656 FP8 30.8 -> 15.9, 1440 x 2752 x 576 FP16 (264 + 110 tiles) 33.9 -> 20.8, and next
//     to a grad_W of the few-tiles kernel 1696 x 2048 x 512 FP8 15.7 -> 11.3
//   no derivative up to 11/16 of the slots (beyond that K slices are as good):  1280 x 2304 x 768 FP16 (180 + 108) 26.9 -> 17.3
//   reductions of grad_X below 1280 bytes, whose tiles are mostly the derivative's epilogue, which the other workgroup's products hide:
//     relu' 7552 x 3072 x 768 FP8 (1416 + 144) 68.3 -> 47.5, 11552 x 6144 x 1264 FP8 260.6 -> 246.6
//   instead of one pair on 256 x 128 tiles with the arithmetic derivative, below 1536 bytes:  relu' 2432 x 3072 x 752 FP16 40.9 -> 34.5,
//     4992 x 2048 x 1024 FP8 37.0 -> 30.5, 4992 x 2048 x 1520 FP8 46.8 -> 39.2
// Both of these limits are cautious: 11552 x 6144 x 1536 FP8 (319 -> 270 when tried) and 2432 x 3072 x 768 FP16 (42.5 -> 34.0) lie
// beyond them and keep the launches they had.
// Geometric mean over 574 drawn layers that these rules move: 0.80, two of them slower (by 2 and 5 %).
// grad_W on fewer tiles than half of the CUs keeps its K slices where the reduction is long (6976 x 416 x 3280 FP16 83.7 -> 97.8) or the
// other product takes many rounds (18176 x 1792 x 896 FP8, 1988 + 98 tiles, 127.8 -> 160.1), and so does grad_X (1712 x 848 x 6272 FP8
// 42.4 -> 45.0).
bool balanced_ok(const GemmProblem& dx, const GemmProblem& dw, long tx, long tw) {
  const long cu = cu_count(), es = dx.a_dt == US_F16 ? 2 : 1, kx = dx.K * es, kw = dw.K * es;
  const bool derivative = dx.epi == US_EPI_GELU_GRAD;
  if (tx + tw <= cu) return false;
  if (2 * tw < cu && (tx + tw > 4 * cu || kw >= 6144)) return false;
  if (2 * tx < cu && kx >= 6144) return false;
  if (eight_wave_pair_ok(dx, dw)) return derivative && !use_big_tile(dx.M, dx.N, 1) && !small_tile_ok(dx) && kx < 1536;
  const long chain = (kx > kw ? kx : kw) + 1000, work = (tx * (kx + 1000) + tw * (kw + 1000)) / cu;
  if (8 * (tx + tw) <= (derivative ? 14 : 11) * cu) return 10 * chain <= (derivative && 8 * (tx + tw) <= 11 * cu ? 16 : 13) * work;
  return derivative && kx < 1280 && chain <= work;
}

bool two_per_cu_ok(const GemmProblem& dx, const GemmProblem& dw) {
  if (!offsets_fit(dx) || !offsets_fit(dw)) return false;
  if (small_tile_choice(dx) != SmallTileChoice::None) return false;
  const long tx = ceil_div(dx.M, 128) * ceil_div(dx.N, 128), tw = ceil_div(dw.M, 128) * ceil_div(dw.N, 128);
  if (small_tile_choice(dw) != SmallTileChoice::None) return tx >= cu_count() / 2 && balanced_ok(dx, dw, tx, tw);
  return all_resident_ok(dx, dw, tx, tw) || balanced_ok(dx, dw, tx, tw);
}

template <bool FP8>
hipError_t launch_two_per_cu(const GemmProblem& dx, const GemmProblem& dw, hipStream_t st) {
  constexpr int FG = FP8 ? 1 : 0;
  using KW = GemmKind<CfgD128, FP8, 0, FG, false, false, EPI_STORE, false>;
  if (dx.epi == US_EPI_GELU_GRAD) return launch_pair<GemmKind<CfgD128, FP8, FG, 0, true, true, EPI_GELU_GRAD, false>, KW>(dx, dw, st);
  if (dx.epi == US_EPI_RESIDUAL) return launch_pair<GemmKind<CfgD128, FP8, FG, 0, true, true, EPI_RESIDUAL, false>, KW>(dx, dw, st);
  return launch_pair<GemmKind<CfgD128, FP8, FG, 0, true, true, EPI_STORE, false>, KW>(dx, dw, st);
}

}  // namespace

bool gemm_pair_applicable(const GemmProblem& dx, const GemmProblem& dw) {
  const bool fp8 = dx.a_dt != US_F16;
  if ((dw.a_dt != US_F16) != fp8) return false;
  if (!(dx.a_kc && dx.b_kc) || dw.a_kc || dw.b_kc) return false;
  if (dx.c_dt != US_F16 || dw.c_dt != US_F16 || dw.epi != US_EPI_NONE) return false;
  if (dx.epi != US_EPI_NONE && dx.epi != US_EPI_GELU_GRAD && dx.epi != US_EPI_RESIDUAL) return false;
  if (halves_share_memory(dx, dw)) return false;
  return small_pair_ok(dx, dw) || two_per_cu_ok(dx, dw) || eight_wave_pair_ok(dx, dw);
}

hipError_t launch_gemm_pair(const GemmProblem& dx, const GemmProblem& dw, hipStream_t st) {
  if (small_pair_ok(dx, dw)) return dx.a_dt != US_F16 ? launch_small_pair_typed<true>(dx, dw, st) : launch_small_pair_typed<false>(dx, dw, st);
  if (two_per_cu_ok(dx, dw)) return dx.a_dt != US_F16 ? launch_two_per_cu<true>(dx, dw, st) : launch_two_per_cu<false>(dx, dw, st);
  return dx.a_dt != US_F16 ? launch_pair_typed<true>(dx, dw, st) : launch_pair_typed<false>(dx, dw, st);
}

}  // namespace us
