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
//      requested behind a store would have to wait for it.
// Measured (one box, forward + backward with the two products for dV and dK): 1024 heads x 128 x 64 148 -> 104 us, 256 heads x
// 512 x 64 328 -> 304 us; timing-only builds of the forward at 512: 102 us as built, 61 without the score stores, 71 with nothing
// but the stores: the two workgroups of a CU run in step, so products and stores overlap only in part.
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
  float scale_s, scale_row, scale_out;
};

// Chunk XOR of a W row: the 32 lanes a transposing read serves together touch 32 bytes in each of the rows r0 .. r0+3 and
// r0+8 .. r0+11; together they must cover all 256 bytes of the banks once.
template <int VP>
__device__ __forceinline__ int swz_w(int row) {
  if (VP == 64) return ((row >> 3) & 1) << 1;
  if (VP == 128) return (((row >> 1) & 1) | (((row >> 3) & 1) << 1)) << 1;
  return ((row & 3) | (((row >> 3) & 1) << 2)) << 1;
}

// fp16(a * f) and fp16(b * f), each product rounded once by a mixed-precision multiply-add.  Its addend is -0, which keeps the
// sign of a zero product, and opaque, or the compiler would fold it away.  (No inline assembly for the multiply itself: its
// operands may come straight from the matrix core, whose result hazards only the compiler's own instructions respect.)
__device__ __forceinline__ int mul_to_half2(float a, float b, float f, float neg_zero) {
  const v2h h = {(_Float16)__builtin_fmaf(a, f, neg_zero), (_Float16)__builtin_fmaf(b, f, neg_zero)};
  return __builtin_bit_cast(int, h);
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
      if (valid && q0 + row < s) wt_store(reinterpret_cast<v8h*>(g.S + hss + (long)(q0 + row) * s + c * 8), v);
      keep[k] = valid ? v : BWD ? zero8 : ninf8;
      x[k] = BWD ? arow[BWD ? p : 0][k] : keep[k];
      top = __builtin_elementwise_max(top, x[k]);
    }
    float m = -__builtin_inff();
#pragma unroll
    for (int q = 0; q < 8; ++q) m = __builtin_fmaxf(m, (float)top[q]);
    m = -kLog2e * group_max<G>(m);
    float sum = 0.0f;
#pragma unroll
    for (int k = 0; k < NCH; ++k)
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        e[k][q] = __builtin_amdgcn_exp2f(__builtin_fmaf((float)x[k][q], kLog2e, m));
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
      __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0): this wave's part of chunk c has landed (nothing else is in flight)
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
        wt_store(reinterpret_cast<v8h*>(g.P + hss + (long)q * s + c * 8),
                 v8h(*US_LDS(const v8h, strip + row * pitch + ((c ^ (row & 15)) << 4))));
    }
  }
}

template <class C, bool BWD>
hipError_t launch(AttnArgs g, hipStream_t st) {
  const int pitch = (2 * g.s + 255) / 256 * 256;
  const int lds = C::BQ * pitch + 2 * C::STAGE;
  static FuncConfig cfg;
  if (hipError_t e = cfg.ensure((const void*)attn_rows_kernel<C, BWD>, 160 * 1024); e != hipSuccess) return e;
  g.nblk = (g.s + C::BQ - 1) / C::BQ;
  // enough heads for every XCD: all blocks of a head on one of them
  const int xcds = device_info().xcds;
  g.by_xcd = g.heads >= 4 * xcds ? xcds : 0;
  const long heads = g.by_xcd ? ((long)g.heads + xcds - 1) / xcds * xcds : g.heads;
  attn_rows_kernel<C, BWD><<<(unsigned)(heads * g.nblk), kThreads, lds, st>>>(g);
  return hipGetLastError();
}

template <bool BWD>
hipError_t dispatch(const AttnArgs& g, hipStream_t st) {
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

bool attention_rows_applicable(bool bwd, const void* X, const void* Y, const void* W, const void* A, const void* S, const void* P,
                               const void* out, long heads, long s, long d) {
  if (s > 2048 || d > 128) return false;
  const size_t nd = (size_t)heads * s * d * 2, ns = (size_t)heads * s * s * 2;
  const void *in[] = {X, Y, W, bwd ? A : nullptr}, *res[] = {S, P, out};
  for (int r = 0; r < 3; ++r) {
    const size_t nr = r < 2 ? ns : nd;
    for (int i = 0; i < 4; ++i)
      if (overlap(in[i], i < 3 ? nd : ns, res[r], nr)) return false;
    for (int q = 0; q < r; ++q)
      if (overlap(res[q], ns, res[r], nr)) return false;
  }
  return true;
}

hipError_t launch_attention_rows(bool bwd, const void* X, const void* Y, const void* W, const void* A, void* S, void* P, void* out,
                                 long heads, long s, long d, float scale_s, float scale_row, float scale_out, hipStream_t st) {
  AttnArgs g{};
  g.X = (const _Float16*)X; g.Y = (const _Float16*)Y; g.W = (const _Float16*)W;
  g.A = (const _Float16*)A;
  g.S = (_Float16*)S; g.P = (_Float16*)P; g.out = (_Float16*)out;
  g.heads = (int)heads; g.s = (int)s; g.d = (int)d;
  g.scale_s = scale_s; g.scale_row = scale_row; g.scale_out = scale_out;
  return bwd ? dispatch<true>(g, st) : dispatch<false>(g, st);
}

}  // namespace us
