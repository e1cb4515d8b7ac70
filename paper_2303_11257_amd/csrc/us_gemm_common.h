// Pieces shared by the two GEMM kernels of the gfx950 library: argument block, tile configuration,
// matrix-core wrappers, workgroup -> tile mapping, and the epilogue that turns a wave's accumulator
// block into scaled FP16 / FP32 rows (optionally through GELU or GELU') with 128-bit global stores.
#pragma once

#include <type_traits>

#include "us_device.h"

namespace us {

// EPI_GELU_TAB / EPI_GELU_GRAD_TAB: same results as EPI_GELU (FP8 activation only) / EPI_GELU_GRAD,
// taken from a table over the FP16 pre-activation that the workgroup copies into LDS.
// EPI_GELU_TAB16: EPI_GELU with an FP16 activation output (and optionally its FP8 copy), from a table.
// EPI_RESIDUAL: C = fp16( skip_scale * R + epi_scale * fp16(scale * acc) ), R an FP16 [M,N] input (Zpre).
enum GemmEpi : int {
  EPI_STORE = 0, EPI_GELU = 1, EPI_GELU_GRAD = 2, EPI_PARTIAL = 3, EPI_GELU_TAB = 4, EPI_GELU_GRAD_TAB = 5, EPI_GELU_TAB16 = 6,
  EPI_RESIDUAL = 7
};

// Division of an unsigned 32-bit number by a divisor that the host knows (Granlund & Montgomery, round-up method): one high
// multiplication and three shifts and additions of scalars, where the compiler's division of two runtime integers is a chain
// of about twenty dependent scalar and vector instructions through a floating-point reciprocal.
struct FastDiv {
  uint32_t mul, pre, post;
  static FastDiv by(uint32_t d) {                                          // 1 <= d < 2^31
    uint32_t l = 0;
    while ((1u << l) < d) ++l;                                             // ceil(log2 d)
    return {(uint32_t)((((uint64_t)1 << 32) * ((1u << l) - d)) / d + 1), l < 1 ? l : 1, l > 1 ? l - 1 : 0};
  }
  __host__ __device__ __forceinline__ uint32_t of(uint32_t n) const {
    const uint32_t t = (uint32_t)(((uint64_t)mul * n) >> 32);
    return (t + ((n - t) >> pre)) >> post;
  }
};

// ---- workgroup -> output tile ------------------------------------------------------------------------
// Workgroups are handed to the device's XCDs round-robin by linear id, and every XCD has its own L2.  When
// the tile grid divides evenly (choose_xcd_grid), XCD x gets a compact rectangle of
// (tiles_m/gm) x (tiles_n/gn) tiles; otherwise the whole grid is one rectangle.  Inside a
// rectangle the tiles are walked in column bands `grp_w` tiles wide, N-fastest within a band, so the
// ~32-64 workgroups that run at the same time on one XCD form a compact block and share the A and B
// panels they stream through that XCD's L2.
// The host prepares the walk: before its first load every workgroup would otherwise do five integer divisions, one behind the
// other, in the largest part of what it spends ahead of its main loop.
struct TileWalk {
  FastDiv by_xcds, by_gm, by_band, by_w, by_last_w;      // by_w: the width of a band, by_last_w: of the last one
  uint32_t xcds, gm, rm, rn, band_tiles, grp_w, last_w, last_band;
  TileWalk() = default;
  // gm = 0: one rectangle
  TileWalk(long tiles_m, long tiles_n, int nxcd, int gm_, int gn, int grp) {
    xcds = gm_ ? (uint32_t)nxcd : 1u;
    gm = gm_ ? (uint32_t)gm_ : 1u;
    rm = (uint32_t)(gm_ ? tiles_m / gm_ : tiles_m);
    rn = (uint32_t)(gm_ ? tiles_n / gn : tiles_n);
    grp_w = (uint32_t)grp;
    band_tiles = rm * grp_w;
    last_band = (rn - 1) / grp_w;
    last_w = rn - last_band * grp_w;
    by_xcds = FastDiv::by(xcds);
    by_gm = FastDiv::by(gm);
    by_band = FastDiv::by(band_tiles);
    by_w = FastDiv::by(grp_w);
    by_last_w = FastDiv::by(last_w);
  }
};

__host__ __device__ __forceinline__ void tile_of_block(const TileWalk& t, uint32_t bid, int& tm, int& tn) {
  const uint32_t idx = t.by_xcds.of(bid), xcd = bid - idx * t.xcds;
  const uint32_t xn = t.by_gm.of(xcd), xm = xcd - xn * t.gm;
  const uint32_t band = t.by_band.of(idx), r = idx - band * t.band_tiles;
  const bool last = band == t.last_band;
  const FastDiv by_w = {last ? t.by_last_w.mul : t.by_w.mul, last ? t.by_last_w.pre : t.by_w.pre, last ? t.by_last_w.post : t.by_w.post};
  const uint32_t q = by_w.of(r);
  tm = (int)(xm * t.rm + q);
  tn = (int)(xn * t.rn + band * t.grp_w + (r - q * (last ? t.last_w : t.grp_w)));
}

// Host side: the split gm x gn = number of XCDs that divides the tile grid and minimises the operand bytes one XCD
// touches (bm, bn: the tile's rows of A and of B); gm = gn = 0 when the grid does not divide.
inline void choose_xcd_grid(long tiles_m, long tiles_n, int nxcd, int bm, int bn, int& gm, int& gn) {
  gm = gn = 0;
  if (nxcd < 2 || (tiles_m * tiles_n) % nxcd != 0) return;
  long best = -1;
  for (int c = 1; c <= nxcd; ++c) {
    if (nxcd % c) continue;
    const int cm = c, cn = nxcd / c;
    if (tiles_m % cm || tiles_n % cn) continue;
    const long cost = tiles_m / cm * bm + tiles_n / cn * bn;     // rows of A plus rows of B that one XCD reads
    if (best < 0 || cost < best) { best = cost; gm = cm; gn = cn; }
  }
}

//   C[M,N] = epilogue( scale * sum_k A(m,k) * B(n,k) )
// An operand is K-contiguous (element (r,k) at base[r*ld + k]) or K-strided (element (r,k) at
// base[k*ld + r]).  What a workgroup needs before its first load comes first, so that it arrives with the first requests to the
// argument segment, which every launch finds cold.
struct GemmArgs {
  const uint8_t* A;
  const uint8_t* B;
  long lda, ldb;         // elements
  long M, N, K;          // K = full reduction length
  long k_per_split;      // reduction range of one slice (blockIdx.y); a multiple of 128 elements
  TileWalk walk;
  void* C;
  long ldc;              // elements
  float scale, epi_scale;
  float skip_scale;      // EPI_RESIDUAL: weight of the skip input
  int act;               // EPI_GELU / EPI_GELU_GRAD (arithmetic forms): which activation, 0 = gelu (us_device.h)
  const _Float16* Zpre;  // EPI_GELU_GRAD: saved pre-activation; EPI_RESIDUAL: skip input; [M,N], leading dimension ldc
  _Float16* aux16;       // EPI_GELU: optional FP16 activation output
  uint8_t* aux8;         // optional FP8 copy of the epilogue's FP16 result
  float* partial;        // EPI_PARTIAL: [splits][M][N] FP32
  const uint8_t* table;  // EPI_*_TAB: the table in global memory (us_device.h)
  long batch_a, batch_b, batch_c;   // bytes between consecutive problems of a batch (blockIdx.z), 0 for a single one
  const _Float16* bias;  // forward product only: optional row [N] added to scale * acc before the rounding, or NULL
  float* colsum;         // EPI_GELU_GRAD / _TAB: optional FP32 [ceil(M / 32)][N], column sums of the FP16 result per 32-row block
};

// Problem number blockIdx.z of a batch of equally shaped, independent products (plain-store epilogue only).
__device__ __forceinline__ void select_batch_item(GemmArgs& g) {
  const long z = blockIdx.z;
  if (z == 0) return;
  g.A += z * g.batch_a;
  g.B += z * g.batch_b;
  g.C = (uint8_t*)g.C + z * g.batch_c;
}

// Tile configuration.  BKB = bytes of K per row and pipeline stage; NST = LDS stage buffers;
// MINB = workgroups per CU the register allocation should allow.  WAVES_K > 1: that many groups of
// WAVES_M x WAVES_N waves work on the same output tile, each on its own share of every stage's k-steps;
// their accumulators are added through LDS before the epilogue (direct kernel only).
template <int BM_, int BN_, int WAVES_M_, int WAVES_N_, int BKB_, int NST_, int MINB_, int WAVES_K_ = 1, bool M16_ = true>
struct GemmCfg {
  // FP16 takes the matrix instructions of 16 x 16 results: next to those of 32 x 32 they move their accumulators half as often, which the
  // power limit turns into clock (random data in registers, nothing else running: 1.92 against 1.65 PFLOP/s).  Not on tiles of few instructions
  // per k-step, nor in short reductions (Short<Cfg>), which the power does not limit and twice as many fragments hold up.
  static constexpr bool M16 = M16_;
  static constexpr int BM = BM_, BN = BN_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, BKB = BKB_, NST = NST_, MINB = MINB_;
  static constexpr int WAVES_K = WAVES_K_;
  static constexpr int WAVES_MN = WAVES_M * WAVES_N;
  static constexpr int WAVES = WAVES_MN * WAVES_K;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  static constexpr int FM = WM / 32, FN = WN / 32;   // 32x32 accumulator blocks per wave
};

#define US_LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

// A wave's accumulators, FM x FN blocks of 32 x 32 results.  The matrix core is fed with the N-side fragment as first operand, so
// a lane ends up with four consecutive columns of one row at a time, four such quads of a block: instructions of 32 x 32 results
// leave quad q at row l%32, column 8q + 4(l/32), those of 16 x 16 at row 16(q/2) + l%16, column 16(q%2) + 4(l/16).
template <int FM, int FN, bool M16>
struct Accumulators {
  using Block = typename std::conditional<M16, v4f, v16f>::type;
  static constexpr int RM = M16 ? 2 * FM : FM, RN = M16 ? 2 * FN : FN;      // rows and columns of instruction results
  static constexpr int COLS = M16 ? 2 : 4;                                  // different quad columns of a block: quad q has column q % COLS
  Block v[RM][RN];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
      for (int j = 0; j < RN; ++j)
#pragma unroll
        for (int r = 0; r < (M16 ? 4 : 16); ++r) v[i][j][r] = 0.0f;
  }
  __device__ __forceinline__ v4f quad(int i, int j, int q) const {
    if constexpr (M16) return v[2 * i + (q >> 1)][2 * j + (q & 1)];
    else return v4f{v[i][j][4 * q], v[i][j][4 * q + 1], v[i][j][4 * q + 2], v[i][j][4 * q + 3]};
  }
  __device__ __forceinline__ void add(int i, int j, int q, v4f x) {
    if constexpr (M16) {
      v[2 * i + (q >> 1)][2 * j + (q & 1)] += x;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[i][j][4 * q + e] += x[e];
    }
  }
  __device__ static __forceinline__ int row(int q, int lane) { return M16 ? 16 * (q >> 1) + (lane & 15) : lane & 31; }
  __device__ static __forceinline__ int col(int q, int lane) { return M16 ? 16 * (q & 1) + 4 * (lane >> 4) : 8 * q + 4 * (lane >> 5); }
};

template <int FA, int FB>
__device__ __forceinline__ v16f mfma_fp8(v8i a, v8i b, v16f c) {
  // format codes of the instruction: 0 = E4M3, 1 = E5M2; unit block scales
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, FA, FB, 0, 0, 0, 0);
}
template <int FA, int FB>
__device__ __forceinline__ v4f mfma_fp8(v8i a, v8i b, v4f c) {
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, FA, FB, 0, 0, 0, 0);
}

__device__ __forceinline__ v16f mfma_f16(v8h a, v8h b, v16f c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ v4f mfma_f16(v8h a, v8h b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }

// Every result leaves through write-through stores (us_device.h).  Measured on the BERT-large step, same box: non-temporal for what
// no kernel reads soon (FP16 / FP32 results of tens of MB) and plain stores for the rest 242 us, write-through for the former only
// 238, for everything 230.5.

// ---- epilogue on a lane's chunks of a strip: eight consecutive columns of one row each (FP16) --------------------------
// What bounds the epilogues of a large tile: the vector ALUs and the latency of the table reads.  An instruction of a wave takes
// a SIMD four cycles, and eight waves with 128 elements per lane each make every instruction per element 0.5 us of a 256 x 256
// tile; fetching their code cold costs as much again where it is tens of KB long.  Hence no bounds check and no address arithmetic
// per access (buffer accesses, below), one instruction per table address, one activation per copy of the code, and the branches
// (rare inputs, optional results) once per strip, so that the reads of all its chunks are in flight together.
// A wave's time in the epilogue (timestamps in the kernel, us, before -> now): relu on 128 x 256 FP8 tiles 9.6 -> 2.8, relu' on
// 128 x 128 7.3 -> 2.8, GELU with an FP16 activation on 256 x 192 11.7 -> 7.7 and, with a bias, on 256 x 256 15.3 -> 9.8, GELU' on
// 256 x 256 FP8 14.7 -> 11.8.  FP8 layer of 2000 x 1552 x 2064 with relu, forward + backward 64.0 -> 53.6.

// byte address of entry number `half HI of w` in a table of 2^SHIFT-byte entries
template <int HI, int SHIFT>
__device__ __forceinline__ uint32_t table_address(uint32_t w) {
  if constexpr (SHIFT == 0) return HI ? w >> 16 : w & 0xffffu;
  uint32_t r;
  const uint32_t n = SHIFT;
  if constexpr (HI)
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "=v"(r) : "v"(n), "v"(w));
  else
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0" : "=v"(r) : "v"(n), "v"(w));
  return r;
}
// LDS by byte address.  The kernels' dynamic LDS is their only LDS and starts at address 0; an address made from the array would
// cost an addition of that 0, which the compiler learns too late.  (A static array would lie in front of it: a test holds the built
// matmul kernels to none.)
template <class T>
__device__ __forceinline__ T lds_read_at(uint32_t a) {
  return *(__attribute__((address_space(3))) const T*)a;
}

typedef unsigned short v2us __attribute__((ext_vector_type(2)));

// E4M3 codes of fp16(alpha_g * gelu(y)) from the byte table at LDS address lut
__device__ __forceinline__ v2i gelu_codes(v8h y, uint32_t lut) {
  const v4i yw = __builtin_bit_cast(v4i, y);
  uint32_t w[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t p = (uint32_t)yw[2 * h], q = (uint32_t)yw[2 * h + 1];
    const v2us even = {lds_read_at<uint8_t>(lut + table_address<0, 0>(p)), lds_read_at<uint8_t>(lut + table_address<0, 0>(q))};
    const v2us odd = {lds_read_at<uint8_t>(lut + table_address<1, 0>(p)), lds_read_at<uint8_t>(lut + table_address<1, 0>(q))};
    w[h] = __builtin_bit_cast(uint32_t, even) | (__builtin_bit_cast(uint32_t, odd) << 8);
  }
  return v2i{(int)w[0], (int)w[1]};
}

// fp16(alpha_g * gelu(y)) for |y| <= 6 from its table; amax collects |y|
__device__ __forceinline__ v8h gelu_halves(v8h y, uint32_t lut, v2us& amax) {
  const v4i yw = __builtin_bit_cast(v4i, y);
  const v2us last = {(unsigned short)kGeluHalfLast, (unsigned short)kGeluHalfLast};
  v4i rw;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const v2us a = __builtin_bit_cast(v2us, yw[q] & 0x7fff7fff);
    amax = __builtin_elementwise_max(amax, a);
    // all ones in the halves that are negative (in assembly: of the four shifts written in C++, ROCm 7.2's compiler emits the
    // first and uses its result four times)
    int neg;
    asm("v_pk_ashrrev_i16 %0, 15, %1 op_sel_hi:[0,1]" : "=v"(neg) : "v"(yw[q]));
    const v2us half = __builtin_bit_cast(v2us, neg & ((kGeluHalfLast + 1) * 0x10001));
    const uint32_t i = __builtin_bit_cast(uint32_t, v2us(half + __builtin_elementwise_min(a, last)));
    const v2us t = {lds_read_at<unsigned short>(lut + table_address<0, 1>(i)), lds_read_at<unsigned short>(lut + table_address<1, 1>(i))};
    rw[q] = __builtin_bit_cast(int, t);
  }
  return __builtin_bit_cast(v8h, rw);
}
// ... and beyond the table: alpha_g * y for positive y (also +inf, NaN), -0 for finite negative y, NaN for -inf
__device__ __forceinline__ v8h gelu_halves_far(v8h y, v8h r, float alpha_g) {
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const uint32_t zb = half_bits(y[k]), a = zb & 0x7fffu;
    float up = alpha_g * (float)y[k];
    asm("" : "+v"(up));                      // two roundings, as in the arithmetic form
    const uint32_t far = (zb & 0x8000u) ? (a >= 0x7c00u ? 0x7e00u : 0x8000u) : half_bits((_Float16)up);
    r[k] = half_from_bits(a > (uint32_t)kGeluHalfLast ? far : half_bits(r[k]));
  }
  return r;
}

// fp16(slope(z) * y), slope = table[|z|] for z >= 0 and beta_g - table[|z|] for z < 0 (FP32), the product rounded once; amax
// collects |z|
__device__ __forceinline__ v8h gelu_gradients(v8h y, v8h z, uint32_t lut, float beta_g, v2us& amax) {
  const v4i yw = __builtin_bit_cast(v4i, y), zw = __builtin_bit_cast(v4i, z);
  const v2us last = {(unsigned short)kGeluSlopeLast, (unsigned short)kGeluSlopeLast};
  v4i rw;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const v2us a = __builtin_bit_cast(v2us, zw[q] & 0x7fff7fff);
    amax = __builtin_elementwise_max(amax, a);
    const uint32_t i = __builtin_bit_cast(uint32_t, v2us(__builtin_elementwise_min(a, last)));    // beyond 8 the slope is exactly beta_g
    float t0 = lds_read_at<float>(lut + table_address<0, 2>(i));
    float t1 = lds_read_at<float>(lut + table_address<1, 2>(i));
    t0 = (short)zw[q] < 0 ? beta_g - t0 : t0;
    t1 = zw[q] < 0 ? beta_g - t1 : t1;
    rw[q] = (int)mul_pair_to_half(t0, t1, (uint32_t)yw[q]);
  }
  return __builtin_bit_cast(v8h, rw);
}

// Sink: c(u, v8h), a16(u, v8h), a8(u, v2i) store chunk u of the matmul result or gradient, the FP16 activation and the FP8 copy.
// y: FP16 matmul results; z: the saved pre-activation (or skip input) at the same positions; lut: LDS address of the table.
// r receives the FP16 result of the GELU' and residual epilogues.
template <int EPI, int AUX_FMT, int ACT, int P, class Sink>
__device__ __forceinline__ void epilogue_chunks(const GemmArgs& g, const Sink& out, const v8h (&y)[P], const v8h (&z)[P], uint32_t lut, v8h (&r)[P]) {
  // the FP16 matmul result itself; forward activations keep it for backward
  if constexpr (EPI == EPI_STORE || EPI == EPI_GELU || EPI == EPI_GELU_TAB || EPI == EPI_GELU_TAB16) {
#pragma unroll
    for (int u = 0; u < P; ++u) out.c(u, y[u]);
  }
  if constexpr (EPI == EPI_STORE) {
    return;
  } else if constexpr (EPI == EPI_GELU_TAB) {
#pragma unroll
    for (int u = 0; u < P; ++u) out.a8(u, gelu_codes(y[u], lut));
    return;
  } else if constexpr (EPI == EPI_GELU_TAB16) {
    v2us amax = {0, 0};
#pragma unroll
    for (int u = 0; u < P; ++u) r[u] = gelu_halves(y[u], lut, amax);
    // inputs beyond the table are rare, so the wave looks for one first
    if (__builtin_amdgcn_ballot_w64(amax.x > (unsigned short)kGeluHalfLast || amax.y > (unsigned short)kGeluHalfLast) != 0) {
#pragma unroll
      for (int u = 0; u < P; ++u) r[u] = gelu_halves_far(y[u], r[u], g.epi_scale);
    }
  } else if constexpr (EPI == EPI_GELU_GRAD_TAB) {
    v2us amax = {0, 0};
#pragma unroll
    for (int u = 0; u < P; ++u) r[u] = gelu_gradients(y[u], z[u], lut, g.epi_scale, amax);
    // +-inf and NaN pre-activations give NaN, as the arithmetic form does: rare, so the wave looks for one first
    if (__builtin_amdgcn_ballot_w64(amax.x >= 0x7c00u || amax.y >= 0x7c00u) != 0) {
#pragma unroll
      for (int u = 0; u < P; ++u)
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if ((half_bits(z[u][k]) & 0x7fffu) >= 0x7c00u) r[u][k] = half_from_bits(0x7e00u);
    }
  } else {
#pragma unroll
    for (int u = 0; u < P; ++u)
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if constexpr (EPI == EPI_RESIDUAL) {
          // weighted addition of the skip input and the FP16-rounded matmul result (the residual layer's
          // interpolation): skip * R rounded to FP32, then one fused multiply-add, then the FP16 rounding
          r[u][k] = to_half(__builtin_fmaf(g.epi_scale, (float)y[u][k], g.skip_scale * (float)z[u][k]));
        } else if constexpr (EPI == EPI_GELU) {
          r[u][k] = to_half(ACT == 0 ? gelu_scaled((float)y[u][k], g.epi_scale) : act_scaled(ACT, (float)y[u][k], g.epi_scale));
        } else {  // EPI_GELU_GRAD: y is the FP16-rounded matmul gradient
          r[u][k] = act_grad_half(ACT, (float)z[u][k], y[u][k], g.epi_scale);
        }
      }
  }
  if constexpr (EPI == EPI_RESIDUAL || EPI == EPI_GELU_GRAD || EPI == EPI_GELU_GRAD_TAB) {
    if (EPI == EPI_RESIDUAL || g.C) {        // a gradient's FP8 copy may be all that is wanted
#pragma unroll
      for (int u = 0; u < P; ++u) out.c(u, r[u]);
    }
  } else if (g.aux16) {
#pragma unroll
    for (int u = 0; u < P; ++u) out.a16(u, r[u]);
  }
  // FP8 copy of the FP16 value just stored: identical to casting the stored tensor afterwards
  if (EPI != EPI_RESIDUAL && g.aux8) {
#pragma unroll
    for (int u = 0; u < P; ++u) out.a8(u, cvt8_fp8_from_half<AUX_FMT>(r[u]));
  }
}

// The activation of the arithmetic epilogues, known where their code is made: f(integral_constant<int, act>).
template <int EPI, class F>
__device__ __forceinline__ void with_activation(const GemmArgs& g, F f) {
  if constexpr (EPI == EPI_GELU || EPI == EPI_GELU_GRAD) {
    if (g.act == 1) f(std::integral_constant<int, 1>{});
    else if (g.act == 2) f(std::integral_constant<int, 2>{});
    else if (g.act == 3) f(std::integral_constant<int, 3>{});
    else f(std::integral_constant<int, 0>{});
  } else {
    f(std::integral_constant<int, 0>{});
  }
}

// Strip geometry: every wave owns 32 rows x WN values of LDS (FP16, or FP32 when WIDE).
template <class Cfg, bool WIDE, int EPI = EPI_STORE>
struct EpiStrip {
  static constexpr int ES = WIDE ? 4 : 2;
  static constexpr int PITCH = Cfg::WN * ES + 16;
  static constexpr int STRIP_BYTES = 32 * PITCH * Cfg::WAVES;
  static constexpr int TABLE_BYTES = EPI == EPI_GELU_TAB ? kGeluTableBytes
                                     : EPI == EPI_GELU_GRAD_TAB ? kGeluSlopeTableBytes
                                     : EPI == EPI_GELU_TAB16 ? kGeluHalfTableBytes : 0;
  static constexpr int BYTES = STRIP_BYTES + TABLE_BYTES;     // the table sits behind the strips
  static constexpr int CPR = Cfg::WN * ES / 16;               // 16-byte chunks per strip row
  static constexpr int PER_LANE = 32 * CPR / 64;              // chunks per lane and strip: numbers lane, lane + 64, ...
  // after PERIOD of them the lanes are back at their columns, RPP rows further down
  static constexpr int PERIOD = 64 % CPR == 0 ? 1 : 3, RPP = PERIOD * 64 / CPR;
  static_assert(PERIOD * 64 % CPR == 0 && PER_LANE % PERIOD == 0, "");
};

constexpr uint32_t kBufferRecords = 0xFFFFFF00u;   // bytes a resource spans; offsets inside a tile stay below (host: offsets_fit)
constexpr uint32_t kOutOfRange = 0xFFFFFFF0u;      // a lane with this offset reads zeros and writes nothing

// Where a lane's chunks lie in a wave's part of a result (or of the saved pre-activation).
template <class S>
struct WaveRows {
  long ld;                     // elements
  int left;                    // rows of the matrix from the wave's first row on (none below 0)
  uint32_t off[S::PERIOD];     // byte offset of this lane's first chunks in a result of S::ES bytes per element
  int row[S::PERIOD], col[S::PERIOD];
  bool in[S::PERIOD];

  __device__ __forceinline__ WaveRows(long ld_, long m, long M, long n, long N, int lane) : ld(ld_) {
    left = __builtin_amdgcn_readfirstlane(M - m > 0x10000 ? 0x10000 : (int)(M - m));
#pragma unroll
    for (int q = 0; q < S::PERIOD; ++q) {
      const int c = lane + q * 64;
      row[q] = c / S::CPR;
      col[q] = c % S::CPR * (16 / S::ES);
      in[q] = n + col[q] < N;
      off[q] = in[q] ? ((uint32_t)row[q] * (uint32_t)ld + (uint32_t)col[q]) * S::ES : kOutOfRange;
    }
  }
};

// One 32-row strip of one tensor.  A buffer resource covers just the rows that exist and a lane whose columns do not exist has an
// offset beyond it, so an access outside the matrix does nothing (a load gives zeros) without a branch, and the rows of a chunk
// are a scalar offset (which the hardware's range check includes): no address arithmetic in the vector ALU.
// LONG: row pitches beyond 32-bit offsets (the register-staged kernel).
template <class S, class T, bool LONG>
struct StripRows {
  static constexpr int ES = sizeof(T);
  const WaveRows<S>& w;
  T* base;                     // first element of the strip
  int left;
  uint32_t bytes;
  __device__ __forceinline__ StripRows(const WaveRows<S>& w_, T* wave_base, int i) : w(w_) {
    base = wave_base + (long)(i * 32) * w.ld;
    left = w.left - i * 32;
    bytes = (uint32_t)__builtin_amdgcn_readfirstlane(left < 0 ? 0 : left < 32 ? left : 32) * (uint32_t)w.ld * ES;
  }
  __device__ __forceinline__ int row0(int u) const { return u / S::PERIOD * S::RPP; }
  __device__ __forceinline__ bool has(int u) const { return w.in[u % S::PERIOD] && row0(u) + w.row[u % S::PERIOD] < left; }
  __device__ __forceinline__ T* at(int u) const { return base + (long)(row0(u) + w.row[u % S::PERIOD]) * w.ld + w.col[u % S::PERIOD]; }
  __device__ __forceinline__ int below(int u) const { return (int)((uint32_t)row0(u) * (uint32_t)w.ld * ES); }
  __device__ __forceinline__ v8h load(int u) const {
    if constexpr (LONG) {
      v8h v = {0, 0, 0, 0, 0, 0, 0, 0};
      if (has(u)) v = *reinterpret_cast<const v8h*>(at(u));
      return v;
    } else {
      return __builtin_bit_cast(v8h, __builtin_amdgcn_raw_buffer_load_b128(
          __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00027000), (int)w.off[u % S::PERIOD], below(u), 0));
    }
  }
  template <class V>
  __device__ __forceinline__ void store(int u, V v) const {
    if constexpr (LONG) {
      if (has(u)) wt_store(reinterpret_cast<V*>(at(u)), v);
    } else if constexpr (sizeof(V) == 8) {
      wt_buffer_store(buffer_words(base, bytes), w.off[u % S::PERIOD] >> 1, below(u), v);           // 8 one-byte elements
    } else {
      wt_buffer_store(buffer_words(base, bytes), w.off[u % S::PERIOD], below(u), __builtin_bit_cast(v4i, v));
    }
  }
};

template <class S, bool LONG>
struct StripSink {
  StripRows<S, _Float16, LONG> C, aux16;
  StripRows<S, uint8_t, LONG> aux8;
  int u0;                      // chunk 0 of the group at hand
  __device__ __forceinline__ StripSink(const GemmArgs& g, const WaveRows<S>& w, long first, int i)
      : C(w, (_Float16*)g.C + first, i), aux16(w, g.aux16 + first, i), aux8(w, g.aux8 + first, i), u0(0) {}
  __device__ __forceinline__ void c(int u, v8h v) const { C.store(u0 + u, v); }
  __device__ __forceinline__ void a16(int u, v8h v) const { aux16.store(u0 + u, v); }
  __device__ __forceinline__ void a8(int u, v2i v) const { aux8.store(u0 + u, v); }
};
// ... and eight columns at element idx of the results
struct PointSink {
  const GemmArgs& g;
  long idx;
  __device__ __forceinline__ void c(int, v8h v) const { wt_store(reinterpret_cast<v8h*>((_Float16*)g.C + idx), v); }
  __device__ __forceinline__ void a16(int, v8h v) const { wt_store(reinterpret_cast<v8h*>(g.aux16 + idx), v); }
  __device__ __forceinline__ void a8(int, v2i v) const { wt_store(reinterpret_cast<v2i*>(g.aux8 + idx), v); }
};

// Each wave pushes 32 rows of its accumulators at a time through its LDS strip and reads them back row-contiguously: all global
// stores (and the read of the saved pre-activation) are 128-bit accesses sweeping whole rows.
// Must be entered after a workgroup barrier (the strips overlay the operand tiles).  A wave works on
// the 32-row blocks I0 .. I1-1 of its accumulators (all of them unless two wave groups share a tile:
// then each group finishes one half of the rows, see the wave-split reduction of the direct kernel).
// BIAS: the kernel is a forward product with an FP16 result and may be given a bias row (GemmArgs::bias); the
// other kernels do not carry the code.
template <bool A_KC, bool B_KC, int EPI, bool WIDE>
constexpr bool epilogue_takes_bias() {
  return A_KC && !B_KC && !WIDE &&
         (EPI == EPI_STORE || EPI == EPI_GELU || EPI == EPI_GELU_TAB || EPI == EPI_GELU_TAB16 || EPI == EPI_RESIDUAL);
}

template <class Cfg, int EPI, bool WIDE, int I0 = 0, int I1 = Cfg::FM, bool BIAS = false, bool LONG = false, class Acc>
__device__ __forceinline__ void store_block_epilogue(const GemmArgs& g, const Acc& acc, uint8_t* lds,
                                                     long m0, long n0, long split) {
  static_assert(WIDE ? (EPI == EPI_STORE || EPI == EPI_PARTIAL) : (EPI != EPI_PARTIAL), "");
  using S = EpiStrip<Cfg, WIDE, EPI>;
  constexpr int AUX_FMT = (EPI == EPI_GELU_GRAD || EPI == EPI_GELU_GRAD_TAB) ? US_E5M2 : US_E4M3;
  static_assert(S::TABLE_BYTES == 0 || Cfg::WAVES_K == 1, "the table copy below meets all waves at a barrier");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int lane = threadIdx.x & 63;
  // Waves whose accumulators take all accumulation registers (128 x 128): a value of its own, or a multiple of the lane's number that the
  // fragment addresses need as well is kept through the main loop, in scratch memory.
  if constexpr (Cfg::FM * Cfg::FN == 16) asm("" : "+v"(lane));
  const int wmn = wave % Cfg::WAVES_MN;
  const long m = m0 + (wmn % Cfg::WAVES_M) * Cfg::WM + I0 * 32;    // first row and column of what this wave stores
  const long n = n0 + (wmn / Cfg::WAVES_M) * Cfg::WN;
  // Bias row: a lane needs the four consecutive values of each of its quad columns.  Requested first, so that the table copy
  // below (where there is one) is in flight at the same time.
  [[maybe_unused]] v4h bias4[BIAS ? Cfg::FN : 1][Acc::COLS] = {};
  [[maybe_unused]] bool has_bias = false;
  if constexpr (BIAS) {
    has_bias = g.bias != nullptr;
    if (has_bias) {
#pragma unroll
      for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
        for (int q = 0; q < Acc::COLS; ++q) {
          const long nb = n + j * 32 + Acc::col(q, lane);
          if (nb < g.N) bias4[j][q] = *reinterpret_cast<const v4h*>(g.bias + nb);
        }
    }
  }
  if constexpr (S::TABLE_BYTES > 0) {
    // copy the table into LDS: whole 1 KB wave loads, 16 bytes per lane, spread over the waves
    for (int c = wave; c < S::TABLE_BYTES / 1024; c += Cfg::WAVES)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(g.table + c * 1024 + lane * 16),
          US_LDS_PTR(void, lds + S::STRIP_BYTES + c * 1024), 16, 0, 0);
  }
  constexpr int EP = S::PITCH;
  uint8_t* strip = lds + wave * (32 * EP);
  const float scale = (EPI == EPI_PARTIAL) ? 1.0f : g.scale;
  constexpr int NI = I1 - I0;                        // 32-row blocks this wave finishes
  const WaveRows<S> rows(EPI == EPI_PARTIAL ? g.N : g.ldc, m, g.M, n, g.N, lane);
  const long first = m * rows.ld + n;
  // GELU' / residual: the second input of the epilogue (saved pre-activation, skip tensor) is requested
  // ahead of its use, for ZGROUP strips at a time and before any store of that group.  Loads and stores
  // share one in-order completion counter here, so a load issued between stores could only be waited for
  // together with every store before it (each one an HBM round trip); GELU' therefore fetches its whole
  // share first and never waits for a store.  The residual epilogue has little arithmetic to hide
  // behind and a tighter register budget (its kernels also hold the wave-split reduction), so it
  // fetches two strips at a time and accepts one store drain in the middle.
  constexpr bool NEEDS_Z = (EPI == EPI_GELU_GRAD || EPI == EPI_GELU_GRAD_TAB || EPI == EPI_RESIDUAL);
  constexpr int ZGROUP = !NEEDS_Z ? 1 : (EPI == EPI_RESIDUAL && NI > 2) ? 2 : NI;
  static_assert(NI % ZGROUP == 0, "");
  v8h zpre[ZGROUP][NEEDS_Z ? S::PER_LANE : 1] = {};
  auto fetch_group = [&](int i0) {
    if constexpr (NEEDS_Z) {
#pragma unroll
      for (int ii = 0; ii < ZGROUP; ++ii) {
        const StripRows<S, const _Float16, LONG> zrows(rows, g.Zpre + first, i0 + ii);
#pragma unroll
        for (int u = 0; u < S::PER_LANE; ++u) zpre[ii][u] = zrows.load(u);
      }
    }
  };
  // Column sums of the FP16 result (the bias gradient of the layer below the activation): a lane always works on
  // the same 8 columns (CPR divides 64), so it adds its rows up in registers; the lanes of a column group are added
  // at the end and the wave writes one FP32 row per 32-row block it finished (the sum in the first, zeros in the
  // others), so that every row of GemmArgs::colsum is written exactly once per column, in an order that is fixed.
  // (Rows beyond the matrix are left out: their row of A is zero, but next to an infinite weight their result is NaN.)
  constexpr bool CAN_COLSUM = (EPI == EPI_GELU_GRAD || EPI == EPI_GELU_GRAD_TAB) && !WIDE && (64 % S::CPR == 0);
  [[maybe_unused]] float cs[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  [[maybe_unused]] bool want_colsum = false;
  if constexpr (CAN_COLSUM) want_colsum = g.colsum != nullptr;
  fetch_group(0);
  with_activation<EPI>(g, [&](auto activation) {
    constexpr int ACT = decltype(activation)::value;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      auto to_strip = [&](auto with_bias) {
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const v4f a = acc.quad(I0 + i, j, q);
            uint8_t* p = strip + Acc::row(q, lane) * EP + (j * 32 + Acc::col(q, lane)) * S::ES;
            if constexpr (WIDE) {
              const v4f o = {a[0] * scale, a[1] * scale, a[2] * scale, a[3] * scale};
              *US_LDS_PTR(v4f, p) = o;
            } else {
              v4h o;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                if constexpr (decltype(with_bias)::value) o[e] = to_half(__builtin_fmaf(a[e], scale, (float)bias4[j][q % Acc::COLS][e]));   // one rounding of the sum
                else o[e] = to_half(a[e] * scale);
              }
              *US_LDS_PTR(v4h, p) = o;
            }
          }
        }
      };
      if constexpr (BIAS) {
        if (has_bias) to_strip(std::true_type{});
        else to_strip(std::false_type{});
      } else {
        to_strip(std::false_type{});
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // one wait for the pre-activation loads, ahead of the stores, which the compiler does not see in the load counter
      if (NEEDS_Z && i % ZGROUP == 0) {
        if (i > 0) fetch_group(i);
        __builtin_amdgcn_s_waitcnt(0x0F70);
      }
      if constexpr (S::TABLE_BYTES > 0) {
        if (i == 0) {      // the table was on its way while the first strip was written
          __builtin_amdgcn_s_waitcnt(0x0F70);
          __syncthreads();
        }
      }
      auto chunk = [&](int u) { return strip + (u / S::PERIOD * S::RPP + rows.row[u % S::PERIOD]) * EP + rows.col[u % S::PERIOD] * S::ES; };
      if constexpr (WIDE) {
        const StripRows<S, float, LONG> wide(
            rows, (EPI == EPI_PARTIAL ? g.partial + (size_t)split * g.M * g.N : (float*)g.C) + first, i);
#pragma unroll
        for (int u = 0; u < S::PER_LANE; ++u) {
          const v4f v = *US_LDS_PTR(const v4f, chunk(u));
          if constexpr (EPI == EPI_PARTIAL) {
            if (wide.has(u)) *reinterpret_cast<v4f*>(wide.at(u)) = v;
          } else {
            wide.store(u, v);
          }
        }
      } else {
        StripSink<S, LONG> sink(g, rows, first, i);
        // all chunks of the strip together, but one by one where the arithmetic needs the registers
        constexpr int GROUP = EPI == EPI_GELU || EPI == EPI_GELU_GRAD ? 1 : S::PER_LANE;
#pragma unroll
        for (int u0 = 0; u0 < S::PER_LANE; u0 += GROUP) {
          v8h y[GROUP], z[GROUP], r[GROUP];
#pragma unroll
          for (int u = 0; u < GROUP; ++u) {
            y[u] = *US_LDS_PTR(const v8h, chunk(u0 + u));
            z[u] = NEEDS_Z ? zpre[NEEDS_Z ? i % ZGROUP : 0][NEEDS_Z ? u0 + u : 0] : y[u];
          }
          sink.u0 = u0;
          epilogue_chunks<EPI, AUX_FMT, ACT>(g, sink, y, z, S::STRIP_BYTES, r);
          if constexpr (CAN_COLSUM) {
            if (want_colsum) {
#pragma unroll
              for (int u = 0; u < GROUP; ++u) {
                if (sink.C.has(u0 + u)) {
#pragma unroll
                  for (int k = 0; k < 8; ++k) cs[k] += (float)r[u][k];
                }
              }
            }
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  });
  if constexpr (CAN_COLSUM) {
    if (want_colsum) {
#pragma unroll
      for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int off = S::CPR; off < 64; off <<= 1) cs[k] += __shfl_xor(cs[k], off, 64);
      const long nc = n + lane * 8;                             // lanes 0 .. CPR-1 hold the wave's WN columns
      const long p0 = m / 32;                                   // first 32-row block this wave finished
      const long prows = (g.M + 31) / 32;
      if (lane < S::CPR && nc < g.N) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          if (p0 + i < prows) {
            float* o = g.colsum + (p0 + i) * g.N + nc;
            const v4f lo = {i == 0 ? cs[0] : 0.0f, i == 0 ? cs[1] : 0.0f, i == 0 ? cs[2] : 0.0f, i == 0 ? cs[3] : 0.0f};
            const v4f hi = {i == 0 ? cs[4] : 0.0f, i == 0 ? cs[5] : 0.0f, i == 0 ? cs[6] : 0.0f, i == 0 ? cs[7] : 0.0f};
            *reinterpret_cast<v4f*>(o) = lo;
            *reinterpret_cast<v4f*>(o + 4) = hi;
          }
        }
      }
    }
  }
}

}  // namespace us
