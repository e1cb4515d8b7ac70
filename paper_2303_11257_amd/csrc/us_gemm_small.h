// GEMM kernel for outputs of few tiles (small batches, small layers): 32 x 32 or 64 x 64 output tiles, so that the tiles
// outnumber the CUs where 128 x 128 tiles would leave most of them idle, and the reduction split over the eight waves of a
// workgroup, so that each wave's chain of stages is an eighth of it.
//
// What bounds it: latency.  Such a product is microseconds of memory traffic at the rate one CU can draw; the time goes into
// the chain load -> LDS -> matrix core -> next stage.  So every wave works alone: it loads its own stages (64 bytes of
// the reduction for all rows of the tile; wave w takes stages w, w + 8, ...; neighbouring waves read neighbouring bytes) into
// its own ring of NST slots, waits only for its own loads, and meets the others once, when the eight partial tiles are added
// through LDS in wave order (FP32, deterministic).  No barrier, no branch in the loop; loads beyond the reduction or the
// matrix are out of range for the buffer resource and return zeros without traffic, so a wave always has NST stages in flight
// and one counted wait fits every iteration.
#pragma once

#include "us_gemm_direct.h"

namespace us {

template <int FM_, int FN_, int NST_>
struct SmallCfg {
  static constexpr int FM = FM_, FN = FN_, NST = NST_;       // 32 x 32 accumulator blocks of the tile; stages per wave
  static constexpr int BM = 32 * FM, BN = 32 * FN, WAVES = 8, THREADS = 64 * WAVES, BKB = 64;
};

template <class Cfg, bool FP8, bool A_KC, bool B_KC>
struct SmallTile {
  static constexpr int ES = FP8 ? 1 : 2;
  static constexpr int BK = Cfg::BKB / ES;
  static constexpr int PA = A_KC ? Cfg::BKB : Cfg::BM * ES, PB = B_KC ? Cfg::BKB : Cfg::BN * ES;
  static constexpr int A_BYTES = Cfg::BM * Cfg::BKB, B_BYTES = Cfg::BN * Cfg::BKB, STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int A_LOADS = A_BYTES / 1024, B_LOADS = B_BYTES / 1024, LOADS = A_LOADS + B_LOADS;   // per wave and stage
  static constexpr int RING_BYTES = Cfg::WAVES * Cfg::NST * STAGE_BYTES;
  // partial tiles: rows of BN + 4 floats, so that 16 lanes at the same column of consecutive rows meet no bank twice
  static constexpr int RP = Cfg::BN + 4;
  static constexpr int REDUCE_BYTES = Cfg::WAVES * Cfg::BM * RP * 4;
  static constexpr int LDS_BYTES = RING_BYTES > REDUCE_BYTES ? RING_BYTES : REDUCE_BYTES;
  static_assert(LDS_BYTES <= 160 * 1024, "");
  static_assert(A_BYTES % 256 == 0 && STAGE_BYTES % 256 == 0, "what direct_frag_f16 asks for");
  static_assert(Cfg::BM * Cfg::BN / 8 <= Cfg::THREADS, "eight results per thread");
};

template <class Cfg, bool FP8, int FA, int FB, bool A_KC, bool B_KC, int EPI, bool WIDE>
__device__ __forceinline__ void gemm_small_tile(const GemmArgs& g, int bid, uint8_t* lds) {
  using T = SmallTile<Cfg, FP8, A_KC, B_KC>;
  constexpr int BM = Cfg::BM, BN = Cfg::BN, FM = Cfg::FM, FN = Cfg::FN, NST = Cfg::NST, W = Cfg::WAVES;
  // FP16: instructions of 16 x 16 results on the smallest tile only (us, layers forward + backward, 16 x 16 -> 32 x 32: 768 x 768 x 768 15.5 -> 15.2,
  // 304 x 512 x 1536 11.3 -> 11.2, 208 x 1536 x 2048 17.5 -> 17.3, 512 x 1024 x 1024 even; on 32 x 32 tiles 32 x 512 x 512 7.06 -> 7.38, 128 x 256 x 256 5.88 -> 5.91)
  constexpr bool M16 = !FP8 && FM * FN == 1;
  constexpr int KSTEPS = FP8 || M16 ? 1 : 2;
  using Acc = Accumulators<FM, FN, M16>;
  constexpr int RM = Acc::RM, RN = Acc::RN, RB = M16 ? 16 : 32;
  int tm, tn;
  tile_of_block(g.walk, (uint32_t)bid, tm, tn);
  const long m0 = (long)tm * BM, n0 = (long)tn * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nstages = (int)((g.K + T::BK - 1) / T::BK);
  uint8_t* ring = lds + wave * (NST * T::STAGE_BYTES);

  OperandLoads<64, BM, Cfg::BKB, A_KC, FP8, T::PA, T::A_LOADS, M16> la;
  OperandLoads<64, BN, Cfg::BKB, B_KC, FP8, T::PB, T::B_LOADS, M16> lb;
  la.init(g.A, g.lda, m0, g.M, (long)wave * T::BK);
  lb.init(g.B, g.ldb, n0, g.N, (long)wave * T::BK);
  const long advA = W * (A_KC ? (long)Cfg::BKB : (long)T::BK * g.lda * T::ES);
  const long advB = W * (B_KC ? (long)Cfg::BKB : (long)T::BK * g.ldb * T::ES);
  long kleft = g.K - (long)wave * T::BK;          // elements of the reduction from the next stage to request on
  auto request = [&](int slot) {
    if (kleft < T::BK) {                          // the last stage, or none: the rest reads zeros from here on
      la.cut((int)kleft);
      lb.cut((int)kleft);
      kleft = 0;
    }
    const __amdgpu_buffer_rsrc_t ra = la.resource(), rb = lb.resource();
    uint8_t* base = ring + slot * T::STAGE_BYTES;
#pragma unroll
    for (int j = 0; j < T::A_LOADS; ++j) la.issue(j, ra, base, 0);
#pragma unroll
    for (int j = 0; j < T::B_LOADS; ++j) lb.issue(j, rb, base + T::A_BYTES, 0);
    la.next += advA;
    lb.next += advB;
    kleft -= W * T::BK;
  };

  Acc acc;
  acc.clear();

#pragma unroll
  for (int s = 0; s < NST; ++s) request(s);
  using FragT = typename std::conditional<FP8, v8i, v8h>::type;
  int slot = 0;
  for (int s = wave; s < nstages; s += W) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * T::LOADS) : "memory");
    FragT fa[KSTEPS][RM], fb[KSTEPS][RN];
    const uint8_t* ta = ring + slot * T::STAGE_BYTES;
    const uint8_t* tb = ta + T::A_BYTES;
#pragma unroll
    for (int k = 0; k < KSTEPS; ++k) {
#pragma unroll
      for (int i = 0; i < RM; ++i) {
        if constexpr (FP8) fa[k][i] = direct_frag_fp8<A_KC, T::PA>(ta, i * RB, k);
        else fa[k][i] = direct_frag_f16<A_KC, T::PA, RM, M16>(ta, 0, i, k);
      }
#pragma unroll
      for (int j = 0; j < RN; ++j) {
        if constexpr (FP8) fb[k][j] = direct_frag_fp8<B_KC, T::PB>(tb, j * RB, k);
        else fb[k][j] = direct_frag_f16<B_KC, T::PB, RN, M16>(tb, 0, j, k);
      }
    }
    lds_reads_done();
#pragma unroll
    for (int k = 0; k < KSTEPS; ++k) {
      frag_ready(fa[k]);
      frag_ready(fb[k]);
    }
    request(slot);
    if (++slot == NST) slot = 0;
#pragma unroll
    for (int k = 0; k < KSTEPS; ++k)
#pragma unroll
      for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RN; ++j) {
          if constexpr (FP8) acc.v[i][j] = mfma_fp8<FB, FA>(fb[k][j], fa[k][i], acc.v[i][j]);
          else acc.v[i][j] = mfma_f16(fb[k][j], fa[k][i], acc.v[i][j]);
        }
  }
  // the zero-filled stages still in flight write LDS that the partial tiles reuse
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // partial tile of this wave
  float* part = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *US_LDS_PTR(v4f, part + (wave * BM + i * 32 + Acc::row(q, lane)) * T::RP + j * 32 + Acc::col(q, lane)) = acc.quad(i, j, q);
  __syncthreads();
  const int row = (int)threadIdx.x / (BN / 8), c8 = (int)threadIdx.x % (BN / 8) * 8;
  const long m = m0 + row, n = n0 + c8;
  constexpr bool NEEDS_Z = EPI == EPI_GELU_GRAD || EPI == EPI_RESIDUAL;
  constexpr bool CAN_COLSUM = EPI == EPI_GELU_GRAD;
  const bool mine = row < BM && m < g.M && n < g.N;
  v8h r = {0, 0, 0, 0, 0, 0, 0, 0};
  if (mine) {
    v8h z = {0, 0, 0, 0, 0, 0, 0, 0}, bias = z;
    if constexpr (NEEDS_Z) z = *reinterpret_cast<const v8h*>(g.Zpre + m * g.ldc + n);
    bool has_bias = false;
    if constexpr (epilogue_takes_bias<A_KC, B_KC, EPI, WIDE>()) {
      has_bias = g.bias != nullptr;
      if (has_bias) bias = *reinterpret_cast<const v8h*>(g.bias + n);
    }
    v4f lo = {0.0f, 0.0f, 0.0f, 0.0f}, hi = lo;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float* p = part + (w * BM + row) * T::RP + c8;
      lo += *US_LDS_PTR(const v4f, p);
      hi += *US_LDS_PTR(const v4f, p + 4);
    }
    if constexpr (WIDE) {
      lo *= g.scale;
      hi *= g.scale;
      wt_store(reinterpret_cast<v4f*>((float*)g.C + m * g.ldc + n), lo);
      wt_store(reinterpret_cast<v4f*>((float*)g.C + m * g.ldc + n + 4), hi);
    } else {
      v8h y;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float a = k < 4 ? lo[k & 3] : hi[k & 3];
        y[k] = to_half(has_bias ? __builtin_fmaf(a, g.scale, (float)bias[k]) : a * g.scale);
      }
      constexpr int AUX_FMT = EPI == EPI_GELU_GRAD ? US_E5M2 : US_E4M3;
      with_activation<EPI>(g, [&](auto activation) {
        const v8h y1[1] = {y}, z1[1] = {z};
        v8h r1[1] = {y};
        epilogue_chunks<EPI, AUX_FMT, decltype(activation)::value>(g, PointSink{g, m * g.ldc + n}, y1, z1, 0, r1);
        r = r1[0];
      });
    }
  }
  if constexpr (CAN_COLSUM) {
    // column sums of the FP16 result per 32-row block (GemmArgs::colsum), rows in order; rows beyond the matrix are zeros
    if (g.colsum != nullptr) {
      __syncthreads();
      _Float16* res = reinterpret_cast<_Float16*>(lds);
      if (row < BM) *US_LDS_PTR(v8h, res + row * BN + c8) = r;
      __syncthreads();
      const int c = (int)threadIdx.x % BN, blk = (int)threadIdx.x / BN;
      if (blk < FM && m0 + blk * 32 < g.M && n0 + c < g.N) {
        float s = 0.0f;
        for (int k = 0; k < 32; ++k) s += (float)*US_LDS_PTR(const _Float16, res + (blk * 32 + k) * BN + c);
        g.colsum[((m0 >> 5) + blk) * g.N + n0 + c] = s;
      }
    }
  }
}

template <class Cfg, bool FP8, int FA, int FB, bool A_KC, bool B_KC, int EPI, bool WIDE>
__global__ void __launch_bounds__(Cfg::THREADS, 1) gemm_small_kernel(GemmArgs g) {
  extern __shared__ __attribute__((aligned(256))) uint8_t lds[];
  gemm_small_tile<Cfg, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(g, (int)blockIdx.x, lds);
}

// grad_X and grad_W of a layer in one launch: the first nb workgroups work on grad_W.
template <class Cfg, bool FP8, int EPI>
__global__ void __launch_bounds__(Cfg::THREADS, 1) gemm_small_pair_kernel(int nb, GemmArgs dx, GemmArgs dw) {
  extern __shared__ __attribute__((aligned(256))) uint8_t lds[];
  constexpr int FG = FP8 ? 1 : 0;                  // format of the gradient operand where it applies (E5M2)
  const int bid = (int)blockIdx.x;
  if (bid < nb) gemm_small_tile<Cfg, FP8, 0, FG, false, false, EPI_STORE, false>(dw, bid, lds);
  else gemm_small_tile<Cfg, FP8, FG, 0, true, true, EPI, false>(dx, bid - nb, lds);
}

}  // namespace us
