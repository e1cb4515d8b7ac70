// Scaled layer norm (Table A.2 "Other"): Y_ij = c_j + w_j (X_ij - mu_i) / sigma_i, alpha = beta_x = 1,
// beta_w = beta_c = b^-1/2.  HBM-bound row kernels: one wave owns a row and keeps it in registers
// (FP16 storage, FP32 arithmetic), so every tensor is read or written exactly once:
//   forward   reads X, writes Y                                   4 B / element
//   backward  reads X and G, writes dX, and leaves per-row-block column sums of G*xhat and G in a
//             workspace; a second small kernel adds the blocks in order (deterministic)      6 B / element
#include "us_launch.h"
#include "us_rows.h"

namespace us {

namespace {

constexpr int kLnThreads = 256;       // four waves, one row each at a time
constexpr int kLnRowsPerBlock = 32;   // fewest rows whose column sums one workgroup accumulates (backward; sizes the scratch)

// mean and 1/sqrt(variance + eps) of the row held in x, zeros beyond n (two passes over the registers)
template <int NCH>
__device__ __forceinline__ void row_stats(const float (&x)[NCH][8], int n, int lane, float eps, float& mean, float& rstd) {
  float s = 0.0f;
#pragma unroll
  for (int k = 0; k < NCH; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) s += x[k][e];
  mean = wave_sum(s) / (float)n;
  float q = 0.0f;
#pragma unroll
  for (int k = 0; k < NCH; ++k) {
    float qk = q;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float d = x[k][e] - mean;
      qk += d * d;
    }
    q = (k * 64 + lane) * 8 < n ? qk : q;
  }
  rstd = 1.0f / __builtin_sqrtf(wave_sum(q) / (float)n + eps);
}

template <int NCH>
__global__ void __launch_bounds__(kLnThreads) ln_fwd_kernel(const _Float16* X, const _Float16* w, const _Float16* c, _Float16* Y,
                                                           long b, int n, float eps) {
  const int lane = threadIdx.x & 63;
  const long wave0 = (long)blockIdx.x * (kLnThreads / 64) + (threadIdx.x >> 6);
  const long nwaves = (long)gridDim.x * (kLnThreads / 64);
  RowRegs<NCH> wr, cr;
  wr.load(w, n, lane);
  cr.load(c, n, lane);
  for (long row = wave0; row < b; row += nwaves) {
    RowRegs<NCH> x;
    x.load(X + row * n, n, lane);
    float xf[NCH][8], mean, rstd;
#pragma unroll
    for (int k = 0; k < NCH; ++k)
#pragma unroll
      for (int e = 0; e < 8; ++e) xf[k][e] = (float)x.v[k][e];
    row_stats<NCH>(xf, n, lane, eps, mean, rstd);
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int col = (k * 64 + lane) * 8;
      if (col < n) {
        v8h o;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          o[e] = to_half(__builtin_fmaf((xf[k][e] - mean) * rstd, (float)wr.v[k][e], (float)cr.v[k][e]));
        wt_store(reinterpret_cast<v8h*>(Y + row * n + col), o);
      }
    }
  }
}

// Backward: dX for kLnRowsPerBlock rows per workgroup, and that block's column sums of G*xhat and G
// into partial[block][2][n] (FP32).  LDS: the waves' sums before they are added in wave order.  The number of workgroups
// is given by the scratch (one per 32 rows), so where a CU gets one or two of them the rows in flight are their NW waves; with
// more, smaller ones share the LDS better.  us, backward (the kernel as it was ahead of the next paragraph; one process) with
// 4 / 8 / 16 waves: 500 x 512 12.0 / 9.8 / 9.2, 8192 x 1024 17.8 / 15.7 / 25.1 (registers), 65536 x 1024 90.4 / 111.7 / 181,
// 65536 x 256 53.8 / 55.4 / 55.3, 4096 x 2048 24.4 / 26.3.
// A row is converted to FP32 once and its registers take the next row at once: no copies, no zeros written again, no values
// spilled in wide rows (30 before); lanes beyond n need no mask where a zero G does the same.  us, backward, before -> this, one process:
// 64 x 2048 22.2 -> 20.4, 2000 x 1008 13.8 -> 13.3, 1500 x 1552 22.4 -> 20.6, 4096 x 768 12.8 -> 12.3, 8192 x 1024 14.9 -> 14.4,
// 65536 x 256 40.4 -> 39.2, 65536 x 1024 89.5 -> 88.7, 32768 x 2048 101.6 -> 93.1, 4096 x 4096 57.5 -> 41.2.
// Every product and every sum is rounded by itself, in the order written, and the number of waves decides which rows are added up
// together: dw holds a few thousand values, so one last place of one of them is already 3e-5 of its norm.  Fused multiply-adds
// (0.4 us of 14.4 at 8192 x 1024) and eight waves for rows of 1032 to 2048 values (20.4 -> 16.4 at 64 x 2048) give other last places: not taken.
template <int NCH, int NW>
__global__ void __launch_bounds__(64 * NW) ln_bwd_kernel(const _Float16* X, const _Float16* w, const _Float16* G, _Float16* dX,
                                                           float* partial, long b, int n, float eps, int rows_per_block) {
  extern __shared__ __attribute__((aligned(16))) float red[];     // [NW waves][2][n]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long row0 = (long)blockIdx.x * rows_per_block;
  RowRegs<NCH> wr;
  wr.load(w, n, lane);
  float aw[NCH][8], ac[NCH][8];
#pragma unroll
  for (int k = 0; k < NCH; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) aw[k][e] = ac[k][e] = 0.0f;
  RowRegs<NCH> x, g;
  if (row0 + wave < b) {
    x.load(X + (row0 + wave) * n, n, lane);
    g.load(G + (row0 + wave) * n, n, lane);
  }
  for (int r = wave; r < rows_per_block; r += NW) {
    const long row = row0 + r, next = row + NW;
    if (row >= b) break;
    float xh[NCH][8], gi[NCH][8];
#pragma unroll
    for (int k = 0; k < NCH; ++k)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        xh[k][e] = (float)x.v[k][e];
        gi[k][e] = (float)g.v[k][e];
      }
    // the next row of this wave is requested into the registers that the current one has just left
    if (r + NW < rows_per_block && next < b) {
#pragma unroll
      for (int k = 0; k < NCH; ++k) {
        const int col = (k * 64 + lane) * 8;
        if (col < n) {
          x.v[k] = *reinterpret_cast<const v8h*>(X + next * n + col);
          g.v[k] = *reinterpret_cast<const v8h*>(G + next * n + col);
        }
      }
    }
    float mean, rstd;
    row_stats<NCH>(xh, n, lane, eps, mean, rstd);
    float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
    for (int k = 0; k < NCH; ++k) {         // (beyond n: gi = 0 adds nothing to the row's sums, and aw and ac are not read)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        xh[k][e] = (xh[k][e] - mean) * rstd;
        ac[k][e] += gi[k][e];
        aw[k][e] += gi[k][e] * xh[k][e];
        gi[k][e] *= (float)wr.v[k][e];
        s1 += gi[k][e];
        s2 += gi[k][e] * xh[k][e];
      }
    }
    const float m1 = wave_sum(s1) / (float)n, m2 = wave_sum(s2) / (float)n;
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int col = (k * 64 + lane) * 8;
      if (col < n) {
        v8h o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = to_half(rstd * (gi[k][e] - m1 - xh[k][e] * m2));
        wt_store(reinterpret_cast<v8h*>(dX + row * n + col), o);
      }
    }
  }
  // the block's column sums: waves in order
#pragma unroll
  for (int k = 0; k < NCH; ++k) {
    const int col = (k * 64 + lane) * 8;
    if (col < n) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        red[(wave * 2 + 0) * n + col + e] = aw[k][e];
        red[(wave * 2 + 1) * n + col + e] = ac[k][e];
      }
    }
  }
  __syncthreads();
  float* out = partial + (size_t)blockIdx.x * 2 * n;
  for (int i = threadIdx.x; i < 2 * n; i += 64 * NW) {
    float s = red[i];
#pragma unroll
    for (int wv = 1; wv < NW; ++wv) s += red[wv * 2 * n + i];
    out[i] = s;
  }
}

// dw_j = beta * sum over blocks of partial[blk][0][j], dc_j likewise from partial[blk][1][j].  A workgroup takes
// 16 of the 2n columns; thread (seg, col) adds the blocks seg, seg + 16, ... (eight independent loads in flight),
// then the 16 segment sums are added in segment order: a fixed association, so the result is reproducible.
__global__ void __launch_bounds__(256) ln_reduce_kernel(const float* partial, _Float16* dw, _Float16* dc, int nblocks, int n,
                                                        float beta) {
  __shared__ float seg_sum[16][17];
  const int col = threadIdx.x & 15, seg = threadIdx.x >> 4;
  const int i = blockIdx.x * 16 + col;               // 0 .. 2n-1 (2n is a multiple of 16)
  const float* p = partial + i;
  const size_t stride = (size_t)2 * n;
  float s = 0.0f;
  int blk = seg;
  for (; blk + 7 * 16 < nblocks; blk += 8 * 16) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(size_t)(blk + u * 16) * stride];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; blk < nblocks; blk += 16) s += p[(size_t)blk * stride];
  seg_sum[seg][col] = s;
  __syncthreads();
  if (seg == 0) {
    float t = seg_sum[0][col];
#pragma unroll
    for (int k = 1; k < 16; ++k) t += seg_sum[k][col];
    const _Float16 o = to_half(beta * t);
    if (i < n) dw[i] = o;
    else dc[i - n] = o;
  }
}

int grid_rows(long b) {
  long g = (b + kLnThreads / 64 - 1) / (kLnThreads / 64);
  if (g > 256 * 16) g = 256 * 16;
  return (int)(g < 1 ? 1 : g);
}

}  // namespace

size_t layer_norm_workspace_bytes(long b, long n) {
  return (size_t)((b + kLnRowsPerBlock - 1) / kLnRowsPerBlock) * 2 * (size_t)n * sizeof(float);
}

hipError_t launch_layer_norm_fwd(const void* X, const void* w, const void* c, void* Y, long b, long n, float eps, hipStream_t st) {
  const _Float16 *x = (const _Float16*)X, *wp = (const _Float16*)w, *cp = (const _Float16*)c;
  _Float16* y = (_Float16*)Y;
  const int nch = (int)((n / 8 + 63) / 64), grid = grid_rows(b);
  if (nch <= 1) ln_fwd_kernel<1><<<grid, kLnThreads, 0, st>>>(x, wp, cp, y, b, (int)n, eps);
  else if (nch <= 2) ln_fwd_kernel<2><<<grid, kLnThreads, 0, st>>>(x, wp, cp, y, b, (int)n, eps);
  else if (nch <= 4) ln_fwd_kernel<4><<<grid, kLnThreads, 0, st>>>(x, wp, cp, y, b, (int)n, eps);
  else ln_fwd_kernel<8><<<grid, kLnThreads, 0, st>>>(x, wp, cp, y, b, (int)n, eps);
  return hipGetLastError();
}

template <int NCH, int NW>
static hipError_t launch_bwd(const _Float16* x, const _Float16* w, const _Float16* g, _Float16* dx, float* partial, long b, int n,
                             float eps, int nblocks, int rows_per_block, hipStream_t st) {
  const int lds = NW * 2 * n * (int)sizeof(float);
  static FuncConfig cfg;
  if (hipError_t e = cfg.ensure((const void*)ln_bwd_kernel<NCH, NW>, 160 * 1024); e != hipSuccess) return e;
  ln_bwd_kernel<NCH, NW><<<nblocks, 64 * NW, lds, st>>>(x, w, g, dx, partial, b, n, eps, rows_per_block);
  return hipGetLastError();
}

hipError_t launch_layer_norm_bwd(const void* X, const void* w, const void* G, void* dX, void* dw, void* dc, long b, long n, float eps,
                                 float beta_wc, void* workspace, hipStream_t st) {
  const _Float16 *x = (const _Float16*)X, *wp = (const _Float16*)w, *g = (const _Float16*)G;
  const int nch = (int)((n / 8 + 63) / 64);
  // at most 4096 workgroups: beyond that each takes more rows (a multiple of the minimum, so the scratch suffices)
  long rpb = kLnRowsPerBlock;
  while ((b + rpb - 1) / rpb > 4096) rpb *= 2;
  const int nblocks = (int)((b + rpb - 1) / rpb);
  float* partial = (float*)workspace;
  hipError_t e;
  const bool few = nblocks <= 2 * device_info().cus;
  if (nch <= 1) e = few ? launch_bwd<1, 16>(x, wp, g, (_Float16*)dX, partial, b, (int)n, eps, nblocks, (int)rpb, st) : launch_bwd<1, 4>(x, wp, g, (_Float16*)dX, partial, b, (int)n, eps, nblocks, (int)rpb, st);
  else if (nch <= 2) e = few ? launch_bwd<2, 8>(x, wp, g, (_Float16*)dX, partial, b, (int)n, eps, nblocks, (int)rpb, st) : launch_bwd<2, 4>(x, wp, g, (_Float16*)dX, partial, b, (int)n, eps, nblocks, (int)rpb, st);
  else if (nch <= 4) e = launch_bwd<4, 4>(x, wp, g, (_Float16*)dX, partial, b, (int)n, eps, nblocks, (int)rpb, st);
  else e = launch_bwd<8, 4>(x, wp, g, (_Float16*)dX, partial, b, (int)n, eps, nblocks, (int)rpb, st);
  if (e != hipSuccess) return e;
  ln_reduce_kernel<<<(unsigned)(2 * n / 16), 256, 0, st>>>(partial, (_Float16*)dw, (_Float16*)dc, nblocks, (int)n, beta_wc);
  return hipGetLastError();
}

}  // namespace us
