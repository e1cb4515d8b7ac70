// Helpers of the row kernels (layer norm, softmax): one wave owns a row of FP16 values and keeps it in
// registers; reductions over the row are cross-lane butterflies with a fixed order of operations.
#pragma once

#include "us_device.h"

namespace us {

// Reductions over groups of G = 16, 32 or 64 lanes; every lane of the group receives the result, in a fixed association.
// The exchanges stay in the vector ALU (DPP inside 16 lanes, row and half swaps beyond): the LDS-permute form of a shuffle
// has several times the latency, and a row kernel with few waves pays it twelve times per row and more (layer norm of 8192 x 1024, forward and
// backward: 27.8 -> 24.1 us; cross-entropy of 8192 x 30528: 216.4 -> 213.0).
template <int CTRL>
__device__ __forceinline__ float lane_dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int G, class F>
__device__ __forceinline__ float group_reduce(float v, F f) {
  static_assert(G == 16 || G == 32 || G == 64, "");
  v = f(v, lane_dpp<0xB1>(v));       // quad_perm [1,0,3,2]: lane ^ 1
  v = f(v, lane_dpp<0x4E>(v));       // quad_perm [2,3,0,1]: lane ^ 2
  v = f(v, lane_dpp<0x141>(v));      // row_half_mirror: the other quad of eight lanes
  v = f(v, lane_dpp<0x140>(v));      // row_mirror: the other half of sixteen lanes
  if constexpr (G >= 32) {           // rows 0 and 1 (2 and 3) of the pair exchange: one result is one row's value, one the other's
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
    const unsigned a = r[0], b = r[1];     // (a bit cast of r[1] itself reads element 0 with this compiler)
    v = f(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
  }
  if constexpr (G == 64) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
    const unsigned a = r[0], b = r[1];     // (a bit cast of r[1] itself reads element 0 with this compiler)
    v = f(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
  }
  return v;
}
template <int G>
__device__ __forceinline__ float group_sum(float v) {
  return group_reduce<G>(v, [](float a, float b) { return a + b; });
}
template <int G>
__device__ __forceinline__ float group_max(float v) {
  return group_reduce<G>(v, [](float a, float b) { return __builtin_fmaxf(a, b); });
}
__device__ __forceinline__ float wave_sum(float v) { return group_sum<64>(v); }
__device__ __forceinline__ float wave_max(float v) { return group_max<64>(v); }

// A wave's reduction by LDS permutes: several times the latency, but hardly any of the vector ALU's time.  For kernels with so many
// waves in flight that the ALU is what they wait for (both forms in one process, us, ALU -> permutes: softmax backward of
// 65536 x 64 22.2 -> 20.7, 131072 x 256 42.4 -> 39.0; cross-entropy of 3490 x 10752 28.0 -> 26.8, but 1100 x 32896 35.4 -> 37.3).
template <class F>
__device__ __forceinline__ float wave_reduce_permute(float v, F f) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = f(v, __shfl_xor(v, off, 64));
  return v;
}
// PERMUTE: which of the two
template <bool PERMUTE>
__device__ __forceinline__ float wave_sum_as(float v) {
  if constexpr (PERMUTE) return wave_reduce_permute(v, [](float a, float b) { return a + b; });
  else return wave_sum(v);
}
template <bool PERMUTE>
__device__ __forceinline__ float wave_max_as(float v) {
  if constexpr (PERMUTE) return wave_reduce_permute(v, [](float a, float b) { return __builtin_fmaxf(a, b); });
  else return wave_max(v);
}

// A row of n FP16 values as NCH chunks of 8 per lane: chunk k of lane l covers columns (k*64 + l)*8 .. +7.
template <int NCH>
struct RowRegs {
  v8h v[NCH];
  __device__ __forceinline__ void load(const _Float16* row, int n, int lane) {
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int col = (k * 64 + lane) * 8;
      if (col < n) v[k] = *reinterpret_cast<const v8h*>(row + col);
      else v[k] = v8h{0, 0, 0, 0, 0, 0, 0, 0};
    }
  }
};

}  // namespace us
