// Attention without mask, the part that works on rows of scores: one kernel per direction, each score row made, normalised,
// stored and used while it is on the chip.
//   forward   S = fp16(sd X Y^T)  (X = Q, Y = K: the scores A)          P = fp16(c softmax(S))               out = fp16(ss P W)  (W = V)
//   backward  S = fp16(sd X Y^T)  (X = dO, Y = V: dP)  dA = fp16(c p (S - sum p S)), p = softmax(A)    out = fp16(ss dA W)  (W = K)
// Every intermediate is rounded to FP16 where the separate calls (two batched products around a softmax kernel) round it, and
// stored, because the next call reads it.
//
// What bounds it: HBM.  The [s, s] tensors are written once (forward: A, P; backward: dP, dA) and A is read once (backward),
// while the separate calls moved them five times forward and six times backward; Q, K, V and the results are 1/8 of that at
// s = 512, d = 64.
//
// A workgroup of 8 waves takes BQ query rows of one head and all s keys.  The BQ x s strip of scores lives in LDS as FP16
// (64 KB at most, so that two workgroups share a CU and one's stores run under the other's products):
//   1. S: the waves split the keys in blocks of 16; X fragments stay in registers, Y fragments come straight from L2 (rows
//      of Y are contiguous along d, which is how the matrix instruction wants them), no barrier in the loop.
//   2. rows: G lanes per row, 16 bytes per lane and chunk, maximum / sum / dot by cross-lane butterflies, FP32 arithmetic; the
//      strip's scores are stored and it becomes P or dA in place.
//   3. out: strip rows times W; W [key][d] is staged through LDS in chunks of KC keys (two buffers, direct-to-LDS loads that
//      read zeros beyond s and d) and transposed on the way to the registers.  The waves split the BQ x d output, and where it
//      has fewer than eight 16 x 16d/2 parts also the keys of a chunk (KS parts, added through LDS in a fixed order).
//   4. P or dA leaves last, with 16-byte stores along the rows: loads and stores share one in-order counter, so a W chunk
//      requested behind a store has to wait for it.  (The scores themselves leave in step 2, ahead of step 3's first wait.)
// Measured, forward + backward with dV and dK, separate steps -> this: 256 heads x 512 x 64 341 -> 276 us back to back on the same
// buffers, 340 -> 274 on inputs that change from pass to pass.  Timing-only builds of the forward at 512, with write-through
// stores: 102 us as built, 61 without the score stores, 71 with nothing but the stores: the two workgroups of a CU run in
// step, so products and stores overlap only in part.
// All times in this file are of calls back to back on the same buffers unless they say otherwise; a kernel trace shows more for
// a single launch (forward at 256 x 512 x 64 116 us, 79 back to back), because it waits until the launch's stores have left.
// LDS layout: 16-byte chunk c of strip row r at c ^ (r & 15) (row pitch a multiple of 256 B), so that the 8-byte writes of step
// 1 and the fragment reads of step 3, 16 rows at the same column each, meet no bank twice; W rows as swz_w() says.
#include "us_device.h"
#include "us_launch.h"
#include "us_rows.h"

namespace us {

namespace {

constexpr int kThreads = 512, kWaves = 8;
constexpr float kLog2e = 1.44269504088896340736f;
#define US_LDS(T, p) ((__attribute__((address_space(3))) T*)(p))

struct AttnArgs {
  const _Float16 *X, *Y, *W;   // [heads, s, d]
  const _Float16* A;           // backward: the stored scores [heads, s, s]
  _Float16 *S, *P, *out;       // forward: A, P, O; backward: dP, dA, dQ
  int heads, s, d, nblk;       // nblk = blocks of BQ query rows per head
  int by_xcd;                  // > 0: the blocks of a head go to one of that many XCDs (they share Y and W in its L2)
  bool stream;                 // the score tensors are larger than what the last-level cache keeps for the next call
  float scale_s, scale_row, scale_out;
};

// 16 bytes of a score tensor.  Written through, a tensor that fits the 256 MB last-level cache is read from there by the next
// call; larger ones only wash the cache, and the non-temporal form writes them faster (us, write-through -> non-temporal, heads x
// s x d, dV and dK still in two launches: forward alone 256 x 512 x 64 112.7 -> 76.8, 64 x 1024 x 64 121 -> 88; forward + backward
// 256 x 512 x 64 309 -> 283, 64 x 1024 x 64 335 -> 280, 128 x 512 x 128 234 -> 219, 512 x 192 x 64 99 -> 109, 1024 x 128 x 64 97 -> 106).
__device__ __forceinline__ void store_scores(bool stream, _Float16* p, v8h v) {
  if (stream) __builtin_nontemporal_store(v, reinterpret_cast<v8h*>(p));
  else wt_store(reinterpret_cast<v8h*>(p), v);
}

// Chunk XOR of a W row: the 32 lanes a transposing read serves together touch 32 bytes in each of the rows r0 .. r0+3 and
// r0+8 .. r0+11; together they must cover all 256 bytes of the banks once.
template <int VP>
__device__ __forceinline__ int swz_w(int row) {
  if (VP == 64) return ((row >> 3) & 1) << 1;
  if (VP == 128) return (((row >> 1) & 1) | (((row >> 3) & 1) << 1)) << 1;
  return ((row & 3) | (((row >> 3) & 1) << 2)) << 1;
}

// ... and of a Y row: 16 lanes read 16 bytes at the same column of the rows 8a + e (+ 4), a, e = 0 .. 3.
template <int VP>
__device__ __forceinline__ int swz_y(int row) {
  if (VP == 64) return (row >> 3) & 3;
  if (VP == 128) return ((row >> 1) & 1) | (((row >> 3) & 3) << 1);
  return (row & 3) | (((row >> 3) & 3) << 2);
}

// s_waitcnt vmcnt(N) alone
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N >= 0 && N < 64, "");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// fp16(a * f) and fp16(b * f), each product rounded once by a mixed-precision multiply-add.  Its addend is -0, which keeps the
// sign of a zero product, and opaque, or the compiler would fold it away.  (No inline assembly for the multiply itself: its
// operands may come straight from the matrix core, whose result hazards only the compiler's own instructions respect.)
__device__ __forceinline__ int mul_to_half2(float a, float b, float f, float neg_zero) {
  const v2h h = {(_Float16)__builtin_fmaf(a, f, neg_zero), (_Float16)__builtin_fmaf(b, f, neg_zero)};
  return __builtin_bit_cast(int, h);
}

// exp(x - m), m the row's maximum, ml = -m log2(e) rounded, rest = m log2(e) + ml.  Forward: one multiply-add; the rounding of ml is a
// factor common to the row, which the normalisation takes out.  Backward: exactly 1 at the maximum, so that the gradient of a row
// whose probability sits on one key, p (dP - sum p dP), cancels to zero; with the common factor it was rounding noise of the
// size of dP s 2^-24.
template <bool BWD>
__device__ __forceinline__ float score_exp(float x, float ml, float rest) {
  const float t = __builtin_fmaf(x, kLog2e, ml);
  return __builtin_amdgcn_exp2f(BWD ? t - rest : t);
}

// BQ query rows per workgroup; rows of at most G * NCH * 8 keys; head size at most 32 * NKS
template <int BQ_, int G_, int NCH_, int NKS_>
struct AttnCfg {
  static constexpr int BQ = BQ_, G = G_, NCH = NCH_, NKS = NKS_;
  static constexpr int QW = BQ / 16, NW = 2, KS = kWaves / (QW * NW);   // waves over query rows, columns of the result, keys
  static constexpr int KC = KS == 4 ? 128 : 64;                         // keys per W chunk: KS * 32 at least
  static constexpr int VP = NKS == 1 ? 64 : NKS == 2 ? 128 : 256;       // pitch of a W row in LDS
  static constexpr int STAGE = KC * VP;
  static constexpr int WLOADS = STAGE / 16;                             // 16-byte loads of a chunk
  static constexpr int LD = (WLOADS + kThreads - 1) / kThreads;         // per thread
  static constexpr int RP = 64 / G, NP = BQ / kWaves / RP;              // rows a wave works on at once, and how often
  static constexpr int MIN_WAVES = BQ == 16 && NKS > 1 ? 2 : 4;         // per SIMD: one workgroup's LDS fills the CU, or two fit
  static_assert(KS >= 1 && KC / 32 >= KS && NP >= 1, "");
  static_assert((KS - 1) * QW * NW * NKS * 1024 <= 2 * STAGE, "the key parts are added in the W buffers");
};

template <class C, bool BWD>
__global__ void __launch_bounds__(kThreads, C::MIN_WAVES) attn_rows_kernel(AttnArgs g) {
  constexpr int BQ = C::BQ, G = C::G, NCH = C::NCH, NKS = C::NKS, KC = C::KC, VP = C::VP, KS = C::KS, NP = C::NP, RP = C::RP;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int s = g.s, d = g.d;
  int head, blk;
  if (g.by_xcd > 0) {
    const int xcd = (int)blockIdx.x % g.by_xcd, i = (int)blockIdx.x / g.by_xcd;
    head = i / g.nblk * g.by_xcd + xcd;
    blk = i % g.nblk;
  } else {
    head = (int)blockIdx.x / g.nblk;
    blk = (int)blockIdx.x % g.nblk;
  }
  if (head >= g.heads) return;
  const int q0 = blk * BQ;
  const int pitch = (2 * s + 255) / 256 * 256;
  uint8_t* strip = lds;
  uint8_t* wbuf = lds + BQ * pitch;
  const long hsd = (long)head * s * d, hss = (long)head * s * s;
  const _Float16 *X = g.X + hsd, *Y = g.Y + hsd;

  // W chunk c (keys c * KC ...) into buffer c & 1
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc((void*)(g.W + hsd), 0, s * d * 2, 0x00027000);
  auto request_w = [&](int c) {
#pragma unroll
    for (int j = 0; j < C::LD; ++j) {
      if (C::WLOADS % kThreads == 0 || wave * 64 + j * kThreads < C::WLOADS) {
        const int o = (j * kThreads + (int)threadIdx.x) * 16;
        const int row = o / VP, chunk = ((o % VP) >> 4) ^ swz_w<VP>(row);
        const int off = chunk * 8 < d ? (c * KC + row) * d * 2 + chunk * 16 : -16;      // beyond the resource: zeros
        __builtin_amdgcn_raw_ptr_buffer_load_lds(wres, US_LDS(void, wbuf + (c & 1) * C::STAGE + (j * kThreads + wave * 64) * 16), 16, off,
                                                 0, 0, 0);
      }
    }
  };
  const int nchunks = (s + KC - 1) / KC;
  request_w(0);
  if (nchunks > 1) request_w(1);

  // ---- 1. scores ----------------------------------------------------------------------------------------------------
  const int l16 = lane & 15, l4 = lane >> 4;
  float neg_zero = -0.0f;
  asm("" : "+v"(neg_zero));
  const v8h zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
  const _Float16 ninf = half_from_bits(0xfc00u);
  const v8h ninf8 = {ninf, ninf, ninf, ninf, ninf, ninf, ninf, ninf};
  v8h xf[BQ / 16][NKS];
#pragma unroll
  for (int r = 0; r < BQ / 16; ++r)
#pragma unroll
    for (int k = 0; k < NKS; ++k) {
      const int q = q0 + r * 16 + l16, col = k * 32 + l4 * 8;
      xf[r][k] = (q < s && col < d) ? *reinterpret_cast<const v8h*>(X + (long)q * d + col) : zero8;
    }
  // backward: the rows of A that step 2 needs are requested now
  const int lg = lane % G, lr = lane / G;
  v8h arow[BWD ? NP : 1][NCH];
  if constexpr (BWD) {
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int k = 0; k < NCH; ++k) {
        const int q = q0 + wave * (BQ / kWaves) + p * RP + lr, col = (k * G + lg) * 8;
        arow[p][k] = (q < s && col < s) ? *reinterpret_cast<const v8h*>(g.A + hss + (long)q * s + col) : ninf8;
      }
  }
  auto load_y = [&](v8h (&yf)[NKS], int kb) {
#pragma unroll
    for (int k = 0; k < NKS; ++k) {
      const int col = k * 32 + l4 * 8;
      yf[k] = col < d ? *reinterpret_cast<const v8h*>(Y + (long)(kb * 16 + l16) * d + col) : zero8;
    }
  };
  auto scores = [&](const v8h (&yf)[NKS], int kb) {
#pragma unroll
    for (int r = 0; r < BQ / 16; ++r) {
      v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int k = 0; k < NKS; ++k) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(yf[k], xf[r][k], acc, 0, 0, 0);
      // register e of lane l: query r*16 + l%16, key kb*16 + 4 (l/16) + e
      const int chunk = (kb * 2 + (l4 >> 1)) ^ l16;
      *US_LDS(v2i, strip + (r * 16 + l16) * pitch + (chunk << 4) + (l4 & 1) * 8) =
          v2i{mul_to_half2(acc[0], acc[1], g.scale_s, neg_zero), mul_to_half2(acc[2], acc[3], g.scale_s, neg_zero)};
    }
  };
  const int nkb = s / 16;
  {
    v8h y0[NKS], y1[NKS];
    int kb = wave;
    if (kb < nkb) load_y(y0, kb);
    for (; kb < nkb; kb += 2 * kWaves) {
      if (kb + kWaves < nkb) load_y(y1, kb + kWaves);
      scores(y0, kb);
      if (kb + 2 * kWaves < nkb) load_y(y0, kb + 2 * kWaves);
      if (kb + kWaves < nkb) scores(y1, kb + kWaves);
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();      // the strip is complete (and the first two W chunks have landed)

  // ---- 2. rows --------------------------------------------------------------------------------------------------------
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int row = wave * (BQ / kWaves) + p * RP + lr;
    // chunks beyond the row hold -inf as scores: they take no part in the maximum and their exponentials are zero
    float e[NCH][8];
    v8h keep[NCH], x[NCH], top = ninf8;      // keep: what the strip holds, the scores (forward) or dP (backward)
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int c = k * G + lg;
      const bool valid = c * 8 < s;
      const v8h v = *US_LDS(const v8h, strip + row * pitch + ((c ^ (row & 15)) << 4));    // (beyond the row: some other LDS)
      if (valid && q0 + row < s) store_scores(g.stream, g.S + hss + (long)(q0 + row) * s + c * 8, v);
      keep[k] = valid ? v : BWD ? zero8 : ninf8;
      x[k] = BWD ? arow[BWD ? p : 0][k] : keep[k];
      top = __builtin_elementwise_max(top, x[k]);
    }
    float m = -__builtin_inff();
#pragma unroll
    for (int q = 0; q < 8; ++q) m = __builtin_fmaxf(m, (float)top[q]);
    m = group_max<G>(m);
    const float ml = -kLog2e * m, rest = __builtin_fmaf(m, kLog2e, ml);
    float sum = 0.0f;
#pragma unroll
    for (int k = 0; k < NCH; ++k)
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        e[k][q] = score_exp<BWD>((float)x[k][q], ml, rest);
        sum += e[k][q];
      }
    sum = group_sum<G>(sum);
    float f, dot = 0.0f;
    if constexpr (BWD) {
      const float inv = 1.0f / sum;
#pragma unroll
      for (int k = 0; k < NCH; ++k)
#pragma unroll
        for (int q = 0; q < 8; ++q) dot = __builtin_fmaf(e[k][q], (float)keep[k][q], dot);
      dot = -inv * group_sum<G>(dot);
      f = g.scale_row * inv;
    } else {
      f = g.scale_row / sum;
    }
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int c = k * G + lg;
      v4i o;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float a = e[k][2 * q], b = e[k][2 * q + 1];
        if constexpr (BWD) {
          a *= (float)keep[k][2 * q] + dot;
          b *= (float)keep[k][2 * q + 1] + dot;
        }
        o[q] = mul_to_half2(a, b, f, neg_zero);
      }
      // the keys between s and the next multiple of 32 take part in step 3: zeros
      if (c * 8 < (s + 31) / 32 * 32) *US_LDS(v4i, strip + row * pitch + ((c ^ (row & 15)) << 4)) = c * 8 < s ? o : v4i{0, 0, 0, 0};
    }
  }
  __syncthreads();

  // ---- 3. result ------------------------------------------------------------------------------------------------------
  const int qw = wave % C::QW, nw = wave / C::QW % C::NW, kp = wave / (C::QW * C::NW);
  v4f acc[NKS];
#pragma unroll
  for (int j = 0; j < NKS; ++j) acc[j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  const uint8_t* prow = strip + (qw * 16 + l16) * pitch;
  for (int c = 0; c < nchunks; ++c) {
    if (c > 0) {
      __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0): this wave's part of chunk c has landed, and step 2's score stores have left
      __builtin_amdgcn_s_barrier();            // everyone's has, and chunk c - 1 is used up
      if (c + 1 < nchunks) request_w(c + 1);
    }
    const uint8_t* wb = wbuf + (c & 1) * C::STAGE;
#pragma unroll
    for (int t = 0; t < KC / 32 / KS; ++t) {
      const int ks = kp * (KC / 32 / KS) + t;              // 32 keys
      if (c * KC + ks * 32 < s) {
        const v8h pf = *US_LDS(const v8h, prow + ((((c * KC + ks * 32) / 8 + l4) ^ l16) << 4));
        v2i w0[NKS], w1[NKS];
        const int krow = ks * 32 + l4 * 8 + (l16 >> 2);
#pragma unroll
        for (int j = 0; j < NKS; ++j) {
          const int chunk = ((nw * NKS + j) * 2 + ((l16 & 3) >> 1)) ^ swz_w<VP>(krow);
          const uint32_t a = (uint32_t)(uintptr_t)US_LDS(const uint8_t, wb + krow * VP + (chunk << 4) + (l16 & 1) * 8);
          asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(w0[j]) : "v"(a));
          asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(w1[j]) : "v"(a), "n"(4 * VP));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int j = 0; j < NKS; ++j) {
          asm volatile("" : "+v"(w0[j]), "+v"(w1[j]));
          const v4i w = {w0[j].x, w0[j].y, w1[j].x, w1[j].y};
          v8h wf;
          __builtin_memcpy(&wf, &w, 16);
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf, pf, acc[j], 0, 0, 0);
        }
      }
    }
  }
  if constexpr (KS > 1) {
    // the key parts, added in their order
    __syncthreads();
    constexpr int MN = C::QW * C::NW;
    const int mn = wave % MN;
    if (kp > 0)
#pragma unroll
      for (int j = 0; j < NKS; ++j) *US_LDS(v4f, wbuf + (((kp - 1) * MN + mn) * NKS + j) * 1024 + lane * 16) = acc[j];
    __syncthreads();
    if (kp == 0)
#pragma unroll
      for (int r = 0; r < KS - 1; ++r)
#pragma unroll
        for (int j = 0; j < NKS; ++j) acc[j] += *US_LDS(const v4f, wbuf + ((r * MN + mn) * NKS + j) * 1024 + lane * 16);
  }
  if (kp == 0) {
    // register e of lane l: query qw*16 + l%16, column n = 4 (l/16) + e of the block
    const int q = q0 + qw * 16 + l16;
#pragma unroll
    for (int j = 0; j < NKS; ++j) {
      const int n = (nw * NKS + j) * 16 + l4 * 4;
      if (q < s && n < d) {
        const v4h o = {to_half(acc[j][0] * g.scale_out), to_half(acc[j][1] * g.scale_out), to_half(acc[j][2] * g.scale_out),
                       to_half(acc[j][3] * g.scale_out)};
        wt_store(reinterpret_cast<v4h*>(g.out + hsd + (long)q * d + n), o);
      }
    }
  }

  // ---- 4. the two score tensors ---------------------------------------------------------------------------------------
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int row = wave * (BQ / kWaves) + p * RP + lr, q = q0 + row;
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int c = k * G + lg;
      if (q < s && c * 8 < s)
        store_scores(g.stream, g.P + hss + (long)q * s + c * 8, v8h(*US_LDS(const v8h, strip + row * pitch + ((c ^ (row & 15)) << 4))));
    }
  }
}

// Rows of at most 128 keys: a wave takes 16 query rows, and their scores never leave its registers.  Keys are the matrix
// instruction's rows, queries its columns, so a lane ends up with scores of one query.  Which key is which row is free: the two
// 16-row products of a 32-key block take keys 8a .. 8a+3 and 8a+4 .. 8a+7, which leaves lane group a with eight consecutive keys:
// 16 bytes of S, and just the operand that step 3 wants.  Step 2 is arithmetic on a lane's values and two lane swaps.
// Y and W pass through LDS as one stream of chunks of KC keys, first those of Y, then those of W (direct-to-LDS loads that read
// zeros beyond s and d): every head's Y and W come cold from memory, a microsecond and more away while the stores of other
// workgroups fill the queues, so all of Y and a chunk of W are requested at once.
// 1024 heads x 128 x 64 with 33.5 MB per score tensor: forward 30.6 -> 26.0 us (4.8 TB/s), backward 62.3 -> 56.5 (both products
// for dV and dK included).  Longer rows the same way (256 keys per wave, 128 registers of scores and exponentials) were slower.
// Head size at most 32 * NKS.
template <int NKS_>
struct AttnShortCfg {
  static constexpr int NB = 4, NKS = NKS_;                              // 32-key blocks of a row
  static constexpr int BQ = 16 * kWaves;                                // query rows per workgroup
  static constexpr int KC = 64;                                         // keys per chunk
  static constexpr int VP = NKS == 1 ? 64 : NKS == 2 ? 128 : 256;       // pitch of a key's row in LDS
  static constexpr int STAGE = KC * VP;
  static constexpr int NBUF = NB / 2 + 1;                               // chunks in LDS: all of Y, and one more
  static constexpr int WLOADS = STAGE / 16;                             // 16-byte loads of a chunk
  static constexpr int LD = (WLOADS + kThreads - 1) / kThreads;         // per thread
  static constexpr int NJ = 2 * NKS;                                    // blocks of 16 columns of the result
  static constexpr int LDS = NBUF * STAGE;
  static constexpr int MIN_WAVES = NKS == 4 ? 2 : 4;                    // per SIMD
};

// maximum / sum over the four lanes that hold parts of one query's row (lanes 16 apart), in a fixed order
template <class F>
__device__ __forceinline__ float quad_rows(float v, F f) {
  const auto p = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
  const unsigned a = p[0], b = p[1];
  v = f(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
  const auto q = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
  const unsigned c = q[0], d = q[1];
  return f(__builtin_bit_cast(float, c), __builtin_bit_cast(float, d));
}

template <class C, bool BWD>
__global__ void __launch_bounds__(kThreads, C::MIN_WAVES) attn_short_rows_kernel(AttnArgs g) {
  constexpr int NB = C::NB, NKS = C::NKS, KC = C::KC, VP = C::VP, NBUF = C::NBUF, NJ = C::NJ;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int s = g.s, d = g.d;
  int head, blk;
  if (g.by_xcd > 0) {
    const int xcd = (int)blockIdx.x % g.by_xcd, i = (int)blockIdx.x / g.by_xcd;
    head = i / g.nblk * g.by_xcd + xcd;
    blk = i % g.nblk;
  } else {
    head = (int)blockIdx.x / g.nblk;
    blk = (int)blockIdx.x % g.nblk;
  }
  if (head >= g.heads) return;
  const int l16 = lane & 15, l4 = lane >> 4;
  const int q = blk * C::BQ + wave * 16 + l16;                            // this lane's query
  const long hsd = (long)head * s * d, hss = (long)head * s * s;
  uint8_t* ring = lds;

  // item t of the stream: chunk t of Y, then chunk t - nchunks of W, into slot t % NBUF
  const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc((void*)(g.Y + hsd), 0, s * d * 2, 0x00027000);
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc((void*)(g.W + hsd), 0, s * d * 2, 0x00027000);
  const int nchunks = (s + KC - 1) / KC, total = 2 * nchunks;
  int fill = 0, use = 0, requested = 0;      // slots of the next item to request and to use
  auto request = [&]() {
    const bool w = requested >= nchunks;
    const int key0 = (w ? requested - nchunks : requested) * KC;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));      // a few instructions each time instead of registers held across the whole kernel
#pragma unroll
    for (int j = 0; j < C::LD; ++j) {
      if (C::WLOADS % kThreads == 0 || wave * 64 + j * kThreads < C::WLOADS) {
        const int o = (j * kThreads + tid) * 16;
        const int row = o / VP, chunk = ((o % VP) >> 4) ^ (w ? swz_w<VP>(row) : swz_y<VP>(row));
        const int off = chunk * 8 < d ? (key0 + row) * d * 2 + chunk * 16 : -16;      // beyond the resource: zeros
        __builtin_amdgcn_raw_ptr_buffer_load_lds(w ? wres : yres, US_LDS(void, ring + fill * C::STAGE + (j * kThreads + wave * 64) * 16), 16,
                                                 off, 0, 0, 0);
      }
    }
    ++requested;
    if (++fill == NBUF) fill = 0;
  };
  // The next item is in LDS for everyone, and the slot of the one before it, which everyone has used up, is filled again.  Of
  // the items requested (two ahead) this wave's part of the next one has landed once only the youngest is in flight; its own
  // reads of the slot have returned before it meets the others.
  static_assert(NBUF == 3, "two items ahead");
  auto advance = [&](int t) {
    if (t + 1 < total) wait_loads<C::LD>();
    else wait_loads<0>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    if (requested < total) request();
    const uint8_t* p = ring + use * C::STAGE;
    if (++use == NBUF) use = 0;
    return p;
  };

  // ---- 1. scores ----------------------------------------------------------------------------------------------------
  float neg_zero = -0.0f;
  asm("" : "+v"(neg_zero));
  const _Float16 ninf = half_from_bits(0xfc00u);
  const v8h ninf8 = {ninf, ninf, ninf, ninf, ninf, ninf, ninf, ninf};
  const v8h zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc((void*)(g.X + hsd), 0, s * d * 2, 0x00027000);
  v8h xf[NKS];
#pragma unroll
  for (int k = 0; k < NKS; ++k) {
    const int col = k * 32 + l4 * 8;
    xf[k] = __builtin_bit_cast(v8h, __builtin_amdgcn_raw_buffer_load_b128(xres, col < d ? (q * d + col) * 2 : -16, 0, 0));
  }
  // first key of this lane's eight in block i, and whether they exist (s is a multiple of 16)
  auto key_of = [&](int i) { return i * 32 + l4 * 8; };
  auto has_keys = [&](int i) { return key_of(i) < s; };
  v8h x[NB];                   // backward: the scores A of this lane's keys
  if constexpr (BWD) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      x[i] = ninf8;
      if (q < s && has_keys(i)) x[i] = *reinterpret_cast<const v8h*>(g.A + hss + (long)q * s + key_of(i));
    }
  }
  __builtin_amdgcn_sched_barrier(0);      // these loads first, the stream behind them
#pragma unroll
  for (int c = 0; c < NBUF - 1; ++c)
    if (c < total) request();
  v8h sc[NB];                  // S of this lane's keys
  const uint8_t* yb = ring;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    sc[i] = BWD ? zero8 : ninf8;
    if (i / 2 < nchunks) {
      if (i % 2 == 0) yb = advance(i / 2);
      v4i o;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int row = (i % 2) * 32 + 8 * (l16 >> 2) + 4 * t + (l16 & 3);
        v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < NKS; ++k) {
          const v8h yf = *US_LDS(const v8h, yb + row * VP + (((k * 4 + l4) ^ swz_y<VP>(row)) << 4));
          acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(yf, xf[k], acc, 0, 0, 0);
        }
        o[2 * t] = mul_to_half2(acc[0], acc[1], g.scale_s, neg_zero);
        o[2 * t + 1] = mul_to_half2(acc[2], acc[3], g.scale_s, neg_zero);
      }
      if (has_keys(i)) sc[i] = __builtin_bit_cast(v8h, o);
    }
  }

  // ---- 2. rows --------------------------------------------------------------------------------------------------------
  // keys beyond the row have -inf as scores: they take no part in the maximum and their exponentials are zero
  if constexpr (!BWD)
#pragma unroll
    for (int i = 0; i < NB; ++i) x[i] = sc[i];
  v8h top = x[0];
#pragma unroll
  for (int i = 1; i < NB; ++i) top = __builtin_elementwise_max(top, x[i]);
  float m = -__builtin_inff();
#pragma unroll
  for (int e = 0; e < 8; ++e) m = __builtin_fmaxf(m, (float)top[e]);
  const auto fmax2 = [](float a, float b) { return __builtin_fmaxf(a, b); };
  const auto add2 = [](float a, float b) { return a + b; };
  m = quad_rows(m, fmax2);
  const float ml = -kLog2e * m, rest = __builtin_fmaf(m, kLog2e, ml);
  float ev[NB][8], sum = 0.0f, dot = 0.0f;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      ev[i][e] = score_exp<BWD>((float)x[i][e], ml, rest);
      sum += ev[i][e];
      if constexpr (BWD) dot = __builtin_fmaf(ev[i][e], (float)sc[i][e], dot);
    }
  sum = quad_rows(sum, add2);
  float f;
  if constexpr (BWD) {
    const float inv = 1.0f / sum;
    dot = -inv * quad_rows(dot, add2);
    f = g.scale_row * inv;
  } else {
    f = g.scale_row / sum;
  }
  v8h pr[NB];                  // P or dA
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    v4i o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float a = ev[i][2 * e], b = ev[i][2 * e + 1];
      if constexpr (BWD) {
        a *= (float)sc[i][2 * e] + dot;
        b *= (float)sc[i][2 * e + 1] + dot;
      }
      o[e] = mul_to_half2(a, b, f, neg_zero);
    }
    pr[i] = has_keys(i) ? __builtin_bit_cast(v8h, o) : zero8;           // keys beyond the row take part in step 3: zeros
  }

  // ---- 3. result ------------------------------------------------------------------------------------------------------
  v4f acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) acc[j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  const uint8_t* wb = ring;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (i / 2 < nchunks) {
      if (i % 2 == 0) wb = advance(nchunks + i / 2);
      v2i w0[NJ], w1[NJ];
      const int krow = (i % 2) * 32 + l4 * 8 + (l16 >> 2);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int chunk = (j * 2 + ((l16 & 3) >> 1)) ^ swz_w<VP>(krow);
        const uint32_t a = (uint32_t)(uintptr_t)US_LDS(const uint8_t, wb + krow * VP + (chunk << 4) + (l16 & 1) * 8);
        asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(w0[j]) : "v"(a));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(w1[j]) : "v"(a), "n"(4 * VP));
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        asm volatile("" : "+v"(w0[j]), "+v"(w1[j]));
        const v4i w = {w0[j].x, w0[j].y, w1[j].x, w1[j].y};
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, w), pr[i], acc[j], 0, 0, 0);
      }
    }
  }
  // register e of lane l: query l%16, column n = 4 (l/16) + e of the block
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int n = j * 16 + l4 * 4;
    if (q < s && n < d) {
      const v4h o = {to_half(acc[j][0] * g.scale_out), to_half(acc[j][1] * g.scale_out), to_half(acc[j][2] * g.scale_out),
                     to_half(acc[j][3] * g.scale_out)};
      wt_store(reinterpret_cast<v4h*>(g.out + hsd + (long)q * d + n), o);
    }
  }

  // ---- 4. the two score tensors ---------------------------------------------------------------------------------------
  if (q < s) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (has_keys(i)) store_scores(g.stream, g.S + hss + (long)q * s + key_of(i), sc[i]);
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (has_keys(i)) store_scores(g.stream, g.P + hss + (long)q * s + key_of(i), pr[i]);
  }
}

// blocks of bq query rows per head; with enough heads for every XCD all blocks of a head go to one of them.  Returns the heads
// that the grid counts.
long spread_over_xcds(AttnArgs& g, int bq) {
  g.nblk = (g.s + bq - 1) / bq;
  const int xcds = device_info().xcds;
  g.by_xcd = g.heads >= 4 * xcds ? xcds : 0;
  return g.by_xcd ? ((long)g.heads + xcds - 1) / xcds * xcds : g.heads;
}

template <class C, bool BWD>
hipError_t launch_short(AttnArgs g, hipStream_t st) {
  static FuncConfig cfg;
  if (hipError_t e = cfg.ensure((const void*)attn_short_rows_kernel<C, BWD>, C::LDS); e != hipSuccess) return e;
  const long heads = spread_over_xcds(g, C::BQ);
  note_gemm_launch("rows", C::BQ, 32 * C::NB, 1, C::NBUF, false, true, true, BWD ? NOTE_SOFTMAX_GRAD : NOTE_SOFTMAX, false, 1);
  attn_short_rows_kernel<C, BWD><<<(unsigned)(heads * g.nblk), kThreads, C::LDS, st>>>(g);
  return hipGetLastError();
}

template <class C, bool BWD>
hipError_t launch(AttnArgs g, hipStream_t st) {
  const int pitch = (2 * g.s + 255) / 256 * 256;
  const int lds = C::BQ * pitch + 2 * C::STAGE;
  static FuncConfig cfg;
  if (hipError_t e = cfg.ensure((const void*)attn_rows_kernel<C, BWD>, 160 * 1024); e != hipSuccess) return e;
  const long heads = spread_over_xcds(g, C::BQ);
  note_gemm_launch("rows", C::BQ, C::G * C::NCH * 8, C::KS, 2, false, true, true, BWD ? NOTE_SOFTMAX_GRAD : NOTE_SOFTMAX, false, 1);
  attn_rows_kernel<C, BWD><<<(unsigned)(heads * g.nblk), kThreads, lds, st>>>(g);
  return hipGetLastError();
}

template <bool BWD>
hipError_t dispatch(const AttnArgs& g, hipStream_t st) {
  // Rows of 65 to 128 keys and at least a workgroup (128 queries) per CU: scores in registers.  Forward + backward, us, strip ->
  // registers, dV and dK on 128 x 128 tiles: 1024 heads x 128 x 64 96.8 -> 84.0 (78 with their narrow tiles, 99.5 on inputs that
  // change from pass to pass), 512 x 128 x 128 87.0 -> 61.3; beside the line 1024 x 64 x 32 34.3 -> 38.5, 64 x 128 x 64 22.3 -> 24.9,
  // 1024 x 256 x 64 (256 keys in registers) 322 -> 385.
  if (g.s > 64 && g.s <= 128 && g.heads >= device_info().cus) {
    if (g.d <= 32) return launch_short<AttnShortCfg<1>, BWD>(g, st);
    return g.d <= 64 ? launch_short<AttnShortCfg<2>, BWD>(g, st) : launch_short<AttnShortCfg<4>, BWD>(g, st);
  }
  // the strip of BQ x s scores takes at most 64 KB; with the W buffers (16 KB up to a head size of 64) two workgroups fit a CU
  if (g.d <= 64) {
    if (g.d <= 32) {
      if (g.s <= 128) return launch<AttnCfg<64, 16, 1, 1>, BWD>(g, st);
      if (g.s <= 256) return launch<AttnCfg<64, 32, 1, 1>, BWD>(g, st);
      if (g.s <= 512) return launch<AttnCfg<64, 64, 1, 1>, BWD>(g, st);
      if (g.s <= 1024) return launch<AttnCfg<32, 64, 2, 1>, BWD>(g, st);
      return launch<AttnCfg<16, 64, 4, 1>, BWD>(g, st);
    }
    if (g.s <= 128) return launch<AttnCfg<64, 16, 1, 2>, BWD>(g, st);
    if (g.s <= 256) return launch<AttnCfg<64, 32, 1, 2>, BWD>(g, st);
    if (g.s <= 512) return launch<AttnCfg<64, 64, 1, 2>, BWD>(g, st);
    if (g.s <= 1024) return launch<AttnCfg<32, 64, 2, 2>, BWD>(g, st);
    return launch<AttnCfg<16, 64, 4, 2>, BWD>(g, st);
  }
  if (g.s <= 128) return launch<AttnCfg<32, 16, 1, 4>, BWD>(g, st);
  if (g.s <= 256) return launch<AttnCfg<32, 32, 1, 4>, BWD>(g, st);
  if (g.s <= 512) return launch<AttnCfg<32, 64, 1, 4>, BWD>(g, st);
  if (g.s <= 1024) return launch<AttnCfg<32, 64, 2, 4>, BWD>(g, st);
  return launch<AttnCfg<16, 64, 4, 4>, BWD>(g, st);
}

}  // namespace

// Whether one kernel is faster than the separate steps.  It always is while launches count and for narrow heads.  With long rows
// or wide heads a workgroup has only 16 or 32 query rows per pass over Y and W, and once the workgroups (w) no longer
// all run at once, the separate products' larger tiles win.  us, separate steps -> rows, both builds in one process or in turn:
//   d = 64   forward 4 / 8 / 12 x 2048 49 -> 37, 70 -> 79, 88 -> 119; 31 / 52 x 1040 78 -> 70, 109 -> 117, 24 x 1280 70 -> 74; backward 16 x 2048 233 -> 247,
//            12 x 2048 192 -> 182;  d = 48 forward 8 / 12 x 2048 66 -> 65, 85 -> 99
//   d = 96   forward 8 / 12 / 24 x 1040 40 -> 36, 44 -> 49, 64 -> 88, 6 / 12 x 1536 43 -> 45, 62 -> 79; 64 x 1024 forward and backward 363 -> 429;
//            backward 12 / 16 x 2048 200 -> 196, 243 -> 296, 24 / 32 x 1280 150 -> 153, 195 -> 230, 32 / 64 x 1024 128 -> 116, 235 -> 280;
//            behind a separate forward 24 / 16 x 1040, x 1280 177 -> 185, 156 -> 157 in all
//   d = 112  forward 4 / 8 x 1040 29 -> 25, 35 -> 39, 3 / 6 x 1536 33 -> 31, 41 -> 47, 16 / 32 x 1024 39 -> 38, 65 -> 72, 128 x 512 66 -> 56;
//            backward 16 x 1040 91 -> 91, 12 x 2048 200 -> 215, 32 / 64 x 1024 126 -> 117, 241 -> 293
//   d = 128  forward 2 / 4 / 8 x 1536 33 -> 23, 37 -> 44, 49 -> 72, 8 / 12 x 1024 29 -> 24, 36 -> 46, 24 / 26 x 640 29 -> 27, 31 -> 39, 23 x 768 34 -> 43;
//            backward 4 / 6 x 1536 78 -> 69, 85 -> 94, 8 / 12 x 1040 78 -> 70, 85 -> 89, 64 x 1024 243 -> 311; behind a separate forward
//            12 / 17 x 1024 100 -> 97, 121 -> 137, 16 / 30 x 832 92 -> 87, 138 -> 154 in all
//            rows of whole 128 x 128 tiles, none of them ragged: forward 200 / 512 x 256 35 -> 42, 78 -> 90, 96 / 148 x 384 41 -> 39, 58 -> 62,
//            32 / 50 x 512 25 -> 21, 32 -> 36, backward 64 / 128 x 512 67 -> 57, 132 -> 136; but 48 x 448, 40 x 528 27 -> 28, 35 -> 33
bool rows_pay(bool bwd, long heads, long s, long d) {
  if (d <= 32) return true;
  const long cu = device_info().cus, bq = s > 1024 ? 16 : s > 512 || d > 64 ? 32 : 64, w = heads * ((s + bq - 1) / bq);
  const long mb = (heads * s * s * 2) >> 20;       // of a score tensor
  if (d <= 64) return bwd ? s <= 1536 || mb <= 96 : s <= 1024 || w * d <= 192 * cu || (s <= 1536 && (d <= 48 || mb <= 72));
  if (d <= 112 && s <= 768) return true;
  if (d <= 112 && s <= 1024 && (bwd || d <= 96)) return mb <= 96;
  if (d <= 96) return 2 * w <= (bwd ? 12 : 5) * cu;
  if (d <= 112) return w <= (bwd ? 4 : 2) * cu;
  if (s > 768) return w <= (bwd ? 2 : 1) * cu;
  if (s > 512) return bwd || w <= 2 * cu;
  if (s <= 128 || s % 128 != 0) return true;
  return mb < (bwd ? 64 : s % 256 != 0 ? 40 : 24);
}

bool attention_rows_applicable(bool bwd, const void* X, const void* Y, const void* W, const void* A, const void* Pf, const void* S,
                               const void* P, const void* out, long heads, long s, long d) {
  if (s > 2048 || d > 128 || !rows_pay(bwd, heads, s, d)) return false;
  const size_t nd = (size_t)heads * s * d * 2, ns = (size_t)heads * s * s * 2;
  const void *in[] = {X, Y, W, bwd ? A : nullptr, bwd ? Pf : nullptr}, *res[] = {S, P, out};
  for (int r = 0; r < 3; ++r) {
    const size_t nr = r < 2 ? ns : nd;
    for (int i = 0; i < 5; ++i)
      if (overlap(in[i], i < 3 ? nd : ns, res[r], nr)) return false;
    for (int q = 0; q < r; ++q)
      if (overlap(res[q], ns, res[r], nr)) return false;
  }
  return true;
}

// dV = P^T dO and dK = dA^T Q leave in one launch behind the rows, while the separate steps make dV first and dK last: neither
// may be written over what the other reads or writes, and dV not over a result of the rows.
bool attention_merged_gradients_ok(const void* Q, const void* P, const void* dO, const void* dP, const void* dA, const void* dQ,
                                   const void* dK, const void* dV, long heads, long s, long d) {
  const size_t nd = (size_t)heads * s * d * 2, ns = (size_t)heads * s * s * 2;
  return !overlap(dV, nd, dP, ns) && !overlap(dV, nd, dA, ns) && !overlap(dV, nd, dQ, nd) && !overlap(dV, nd, Q, nd) &&
         !overlap(dV, nd, dK, nd) && !overlap(dK, nd, P, ns) && !overlap(dK, nd, dO, nd);
}

hipError_t launch_attention_rows(bool bwd, const void* X, const void* Y, const void* W, const void* A, void* S, void* P, void* out,
                                 long heads, long s, long d, float scale_s, float scale_row, float scale_out, hipStream_t st) {
  AttnArgs g{};
  g.X = (const _Float16*)X; g.Y = (const _Float16*)Y; g.W = (const _Float16*)W;
  g.A = (const _Float16*)A;
  g.S = (_Float16*)S; g.P = (_Float16*)P; g.out = (_Float16*)out;
  g.heads = (int)heads; g.s = (int)s; g.d = (int)d;
  g.stream = heads * s * s * 2 >= 64l << 20;       // a step writes four score tensors: A, P, dP, dA
  g.scale_s = scale_s; g.scale_row = scale_row; g.scale_out = scale_out;
  return bwd ? dispatch<true>(g, st) : dispatch<false>(g, st);
}

}  // namespace us
