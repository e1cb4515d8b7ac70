// Direct-to-LDS pipelined GEMM kernel for gfx950 (every shape whose tiles span less than 4 GB of an operand).
//
// Operand tiles travel HBM/L2 -> LDS with buffer_load_dwordx4 ... lds (no register staging, no LDS store instructions): a
// wave instruction deposits 64 x 16 B contiguously, so tiles are unpadded and bank conflicts are removed by an XOR swizzle
// of the 16-byte chunk index instead; the swizzle is applied to the *global* offset each lane fetches and again when
// fragments are read.  A buffer resource starts at the tile's first row and moves along the reduction with the stages
// (scalar arithmetic only); a lane keeps one 32-bit offset per load for the whole main loop.  Rows beyond the matrix and the
// part of the last stage beyond the reduction length get an offset that the hardware's range check turns into zeros, so
// every lane of every load is always active: ragged tiles and ragged reduction lengths run the same loop, and the number
// of loads in flight is a constant that the counted waits below rely on.
// (Before: 64-bit global addresses, a null check and an exec mask per load, ~60 vector and ~60 scalar instructions and 16
// branches per stage around the 16 matrix instructions of the 256 x 256 tile, now 24, 35 and one.  One box, both builds in
// turn: 64-token FP8 inference 42.9 -> 32.1 us, attention of 1024 heads x 128 157 -> 148, BERT-large FP8 step 243.5 -> 238.7,
// FP16 BERT-base 173.2 -> 169.5; the 32768 x 4096 x 16384 step, held back by power, unchanged at 10.8 ms.  Ragged reductions
// leave the register-staged kernel: FP16 FFN of 4016 x 1008 x 4000 with biases 391 -> 266 us.)
// NST stage buffers form a ring.  Matrix-core fragments are double-buffered in registers (FP8 with 128 bytes of k per wave and stage: one
// set, requested again piece by piece, KStep128): the LDS reads of
// the next k-step are issued one fragment at a time behind the later MFMAs of the current one, also across the stage boundary.  At that boundary a wave waits for its own LDS reads of
// stage s, then for its own loads of stage s+1 (explicit s_waitcnt vmcnt(n): younger stages stay in flight), then meets the
// other waves at one bare s_barrier; after it the buffer of stage s is free and receives the loads
// of stage s+NST, so NST stages of HBM latency are covered by MFMAs.  The loop runs branch-free while there is a stage
// to refill; the last NST stages are a second copy of the body without loads.
//
// Tile layouts in LDS (pitch P bytes, chunk = 16 B, c' = c ^ swz(row)):
//   K-contiguous operand: [row][BKB bytes]        fragments: ds_read_b128
//   K-strided operand:    [k][rows * elem size]   fragments: ds_read_b64_tr_b8 / _tr_b16 (transposing)
#pragma once

#include <type_traits>
#include <utility>

#include "us_gemm_common.h"

namespace us {

template <class Cfg, bool FP8, bool A_KC, bool B_KC, bool WIDE, int EPI = EPI_STORE>
struct DirectTile {
  static constexpr int ES = FP8 ? 1 : 2;
  static constexpr int BK = Cfg::BKB / ES;                      // elements of K per stage
  static constexpr int PA = A_KC ? Cfg::BKB : Cfg::BM * ES;     // LDS pitch of the A / B tile
  static constexpr int PB = B_KC ? Cfg::BKB : Cfg::BN * ES;
  static constexpr int A_BYTES = Cfg::BM * Cfg::BKB;
  static constexpr int B_BYTES = Cfg::BN * Cfg::BKB;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int A_LOADS = A_BYTES / 16 / Cfg::THREADS;   // 16-byte loads per thread and stage
  static constexpr int B_LOADS = B_BYTES / 16 / Cfg::THREADS;
  // FP8: instructions of 16 x 16 results over 128 k where a wave's share of a stage is 128 bytes of k (main loop below), but not on waves of 64 x 64 that
  // take all of a stage's k (D128, H256): with 16 instructions a stage, of which the boundary lies behind eight, the refill has too little time.  With / without,
  // 51 products of 192 to 376 tiles: K = 512 1.04 to 1.09 in every layout; 1024 to 2048 forward 0.98 to 1.08, grad_W 1.01 to 1.04, grad_X 0.97 to 0.99; from 3072 on
  // 0.94 to 1.00, but 1.02 where a few tiles are alone in the last round (992 x 6000); layers, forward and backward, 0.98 to 1.00.
  static constexpr bool K128 = FP8 && Cfg::M16 && Cfg::BKB == 128 * Cfg::WAVES_K && (Cfg::FM * Cfg::FN > 4 || Cfg::WAVES_K > 1);
  static constexpr bool M16 = FP8 ? K128 : Cfg::M16;            // matrix instructions of 16 x 16 results
  static constexpr int RING_BYTES = Cfg::NST * STAGE_BYTES;
  // WAVES_K = 2: the half of every wave's accumulators that its partner finishes (FP32, one 256-byte row
  // per register) passes through LDS before the strips take the same space
  static constexpr int REDUCE_BYTES = Cfg::WAVES_K == 1 ? 0 : Cfg::WAVES * (Cfg::FM / 2) * Cfg::FN * 16 * 64 * 4;
  static constexpr int STRIP_TABLE_BYTES = EpiStrip<Cfg, WIDE, EPI>::BYTES;
  static constexpr int EPI_BYTES = REDUCE_BYTES > STRIP_TABLE_BYTES ? REDUCE_BYTES : STRIP_TABLE_BYTES;
  static constexpr int LDS_BYTES = RING_BYTES > EPI_BYTES ? RING_BYTES : EPI_BYTES;
  static_assert(A_BYTES % (16 * Cfg::THREADS) == 0 && B_BYTES % (16 * Cfg::THREADS) == 0, "whole wave loads only");
  static_assert(Cfg::NST >= 2 && Cfg::NST <= 5, "");
  static_assert(Cfg::BKB == 64 || Cfg::BKB == 128 || (Cfg::BKB == 256 && !A_KC && !B_KC),
                "256-byte stages exist for K-strided tiles only (the K-contiguous swizzle stops at 128)");
  static_assert(Cfg::BKB / 64 % Cfg::WAVES_K == 0, "whole k-steps per wave group");
  static_assert(LDS_BYTES <= 160 * 1024, "the ring must fit the CU's 160 KB of LDS");
  // The fragment addresses of K128 (Frags128) flip bits of an LDS address: the chunk index of a fragment's rows has to be a field of its own in
  // it, of a power of two of fragments from the wave's first one on, above tiles that start at a multiple of 128 bytes.
  static constexpr bool power_of_two(int n) { return (n & (n - 1)) == 0; }
  static_assert(!K128 || ((A_KC || power_of_two(Cfg::FM)) && (B_KC || power_of_two(Cfg::FN))), "K-strided fragments of K128: a power of two per wave");
  static_assert(!K128 || (A_BYTES % 128 == 0 && STAGE_BYTES % 128 == 0 && 2 * Cfg::FM * 16 <= 128 && 2 * Cfg::FN * 16 <= 128), "tiles of K128 start at 128 bytes");
  // ... and the numbers of up to eight K-strided FP16 fragments (direct_frag_f16)
  static_assert(FP8 || (A_BYTES % 256 == 0 && STAGE_BYTES % 256 == 0 && Cfg::FM <= 4 && Cfg::FN <= 4), "tiles of FP16 start at 256 bytes");
};

// XOR mask on the 16-byte chunk index of LDS row `row`, chosen so that the fragment reads below are free of
// bank conflicts (64 banks x 4 B; b64 reads are served 32 lanes at a time, b128 reads 16: lanes 0-3, 12-15, 20-27, then 4-11, 16-19, 28-31,
// and the same of the upper half).  M16: fragments of the 16 x 16 instructions.
// K-contiguous, the eight (pitch 128) row pairs or four (64) row quads of 16 rows differ in their mask: 16 lanes that read one chunk of 16 different rows
// cover the banks.  Of 16-row fragments they read rows of two k-quarters, in each other's places.  The second quarter's chunk is one further in
// FP16, which the pitch of 128 takes as it is (that of 64, few tiles, has two lanes at a bank; masks without that were slower there as often as
// faster).  In FP8 it is two further, so the masks of the row pairs 0, 1, 6, 7 have to be closed under a flip of bit 1: 0 to 3.  (With the plain number
// of the row pair as mask, 256 x 256 tiles spent 64 more conflict cycles per wave and stage; us before -> now: NT 6000 x 4096, K = 16 13.5 -> 13.2, K = 256
// 16.1 -> 15.7, K = 1024 28.4 -> 27.8; NN 8192 x 4096, K = 16 16.1 -> 15.9, K = 768 28.4 -> 28.1.)
// M16 FP8, K-strided: 16 rows x 128 k, whose 32 lanes read two blocks of eight k-rows, 32 apart, of the same columns (of 32
// rows x 64 k: neighbouring columns of one block); bit 5 of the k-row sends the second one to the other half of the banks.
template <bool KC, bool FP8, int PITCH, bool M16>
__host__ __device__ constexpr int swz(int row) {
  if constexpr (KC) {
    static_assert(PITCH == 64 || PITCH == 128, "K-contiguous pitch");
    const int p = PITCH == 64 ? (row >> 2) & 3 : (row >> 1) & 7;
    return M16 && FP8 ? p ^ (p << 1 & 4) : p;
  } else if constexpr (FP8) {
    static_assert(PITCH == 32 || PITCH == 64 || PITCH == 128 || PITCH == 256, "K-strided FP8 pitch");
    // (eight k-rows of 32 B in a row cover the banks as they are; of 64 B, rows 0-3 and 4-7 take different halves)
    static_assert(!M16 || PITCH >= 128, "");
    return (PITCH == 32 ? 0 : PITCH == 64 ? (((row >> 2) & 1) << 1) : PITCH == 256 ? ((row & 7) << 1) : (((row >> 1) & 3) << 1)) |
           (M16 ? (row >> 5) & 1 : 0);
  } else {
    static_assert(PITCH == 64 || PITCH == 128 || PITCH == 256 || PITCH == 384 || PITCH == 512, "K-strided FP16 pitch");
    // 32-row fragments: the 32 lanes a transposing read serves together touch 64 contiguous bytes in each of four consecutive k-rows, and the same
    // goes for each of those moving by a different multiple of 64 B, or for one bit of it.
    if constexpr (!M16) return PITCH == 64 ? 0 : PITCH == 128 || PITCH == 384 ? ((row >> 1) & 1) << 2 : (row & 3) << 2;
    // 16-row fragments: they touch 32 contiguous bytes in each of the k-rows r .. r+3 and r+8 .. r+11.
    // Pitches of 256 / 512 B put those rows on the same banks: each of the eight moves by a different multiple of 32 B.  Pitches of
    // 128 and 384 B (a tile 192 values wide) already alternate between two bank halves, of 64 B between four quarters, so two bits or
    // one are left (they stay inside a row of 384 B: 24 chunks are three groups of eight).
    return PITCH == 64 ? ((row >> 3) & 1) << 1
           : PITCH == 128 || PITCH == 384 ? (((row >> 1) & 1) | (((row >> 3) & 1) << 1)) << 1
                                          : ((row & 3) | (((row >> 3) & 1) << 2)) << 1;
  }
}

// Byte offset in a K-contiguous tile of the first 16 bytes that lane l reads of the fragment of its first rows, k-step `kstep` of the stage; other
// fragments, whole multiples of 16 rows further down, have the same masks and lie a constant away.  FP8 lanes read the next chunk as well: the offset
// with bit 4 flipped.
template <bool FP8, int PITCH, bool M16>
__host__ __device__ constexpr int kc_fragment(int l, int kstep) {
  constexpr int LOG_ROWS = M16 ? 4 : 5, CHUNKS = FP8 ? 2 : 1;
  const int r = l & ((1 << LOG_ROWS) - 1), c = (kstep * (64 >> LOG_ROWS) + (l >> LOG_ROWS)) * CHUNKS;
  return r * PITCH + ((c ^ swz<true, FP8, PITCH, M16>(r)) << 4);
}

// The same of a K-strided FP16 tile (`pitch` bytes per k-row) and the fragment whose first row is r0: 16 lanes cooperate on a 4(k) x 16(row) block of
// halves, lane i points at k-row i/4, row quarter i%4, and receives the 4 k values of row (group base + i); the second read is 4 k-rows further down.
template <int PITCH, bool M16>
__host__ __device__ constexpr int ks_fragment_f16(int l, int r0, int kstep) {
  const int krow = (M16 ? kstep * 32 + (l >> 4) * 8 : kstep * 16 + (l >> 5) * 8) + ((l & 15) >> 2);
  const int colb = (r0 + (M16 ? 0 : (l >> 4 & 1) * 16) + (l & 3) * 4) * 2;
  return krow * PITCH + (((colb >> 4) ^ swz<false, false, PITCH, M16>(krow)) << 4) + (colb & 15);
}

// One operand's loads: NL 16-byte loads per thread and stage of a tile of ROWS rows.
template <int THREADS, int ROWS, int BKB, bool KC, bool FP8, int PITCH, int NL, bool M16>
struct OperandLoads {
  static constexpr int ES = FP8 ? 1 : 2;
  uint32_t off[NL];            // byte offset of this lane's chunk from (first row, first k of the stage)
  const uint8_t* next;         // wave-uniform: (first row, first k) of the next stage to request

  // THREADS: the threads that load the tile together, the whole workgroup or one wave
  __device__ static __forceinline__ int lds_row(int j) { return (j * THREADS + ((int)threadIdx.x & (THREADS - 1))) * 16 / PITCH; }
  __device__ static __forceinline__ int chunk(int j) {
    if (KC && THREADS * 16 % (16 * PITCH) == 0) j = 0;       // whole multiples of 16 rows apart: the same masks
    const int o = (j * THREADS + ((int)threadIdx.x & (THREADS - 1))) * 16;
    return ((o % PITCH) >> 4) ^ swz<KC, FP8, PITCH, M16>(o / PITCH);
  }
  __device__ __forceinline__ void init(const uint8_t* base, long ld, long row0, long extent_r, long k0) {
    next = base + (KC ? row0 * ld + k0 : k0 * ld + row0) * ES;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int r = KC ? lds_row(j) : chunk(j) * (16 / ES);
      off[j] = (row0 + r < extent_r) ? (uint32_t)lds_row(j) * (uint32_t)(ld * ES) + (uint32_t)chunk(j) * 16u : kOutOfRange;
    }
  }
  // the last stage holds only `krem` elements of the reduction
  __device__ __forceinline__ void cut(int krem) {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int k = KC ? chunk(j) * (16 / ES) : lds_row(j);
      if (k >= krem) off[j] = kOutOfRange;
    }
  }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t resource() const {
    return __builtin_amdgcn_make_buffer_rsrc((void*)next, 0, (int)kBufferRecords, 0x00027000);
  }
  // load j of a stage into the tile at `tile`: lane l of wave w lands at (j * THREADS + 64 w + l) * 16
  __device__ __forceinline__ void issue(int j, __amdgpu_buffer_rsrc_t r, uint8_t* tile, int wave) const {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, US_LDS_PTR(void, tile + (j * THREADS + wave * 64) * 16), 16, (int)off[j], 0, 0, 0);
  }
};

// LDS byte address of a pointer into the workgroup's LDS allocation.
__device__ __forceinline__ uint32_t lds_addr(const uint8_t* p) {
  return (uint32_t)(uintptr_t)US_LDS_PTR(const uint8_t, p);
}

// The transposing LDS reads are issued through inline assembly: the compiler cannot see what they
// read and would otherwise order them after ALL pending direct-to-LDS loads (s_waitcnt vmcnt(0)),
// which would serialise the pipeline.  It therefore does not count them either: every consumer of a
// fragment first passes through frag_ready() below.
template <int OFFSET>
__device__ __forceinline__ v2i ds_read_tr8(uint32_t addr) {
  v2i v;
  asm volatile("ds_read_b64_tr_b8 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFFSET));
  return v;
}
template <int OFFSET>
__device__ __forceinline__ v2i ds_read_tr16(uint32_t addr) {
  v2i v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFFSET));
  return v;
}
// Wait for every LDS read issued so far and tie the fragment registers to that wait, so that no use
// of them can be scheduled above it.
__device__ __forceinline__ void lds_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
template <class F, int N>
__device__ __forceinline__ void frag_ready(F (&f)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(f[i]));
}

// Fragment = the 32 (r0 .. r0+31) or 16 (M16) rows of one MFMA x its k, number `kstep` within the stage: 64 bytes, FP16 of 32 rows 32.  Lane l
// supplies 32 (FP8) or 8 (FP16) consecutive k of one row: of row r0 + l%32 those of k-half l/32, or of row r0 + l%16 those of k-quarter l/16.
template <bool KC, int PITCH>
__device__ __forceinline__ v8i direct_frag_fp8(const uint8_t* tile, int r0, int kstep) {
  const int l = threadIdx.x & 63;
  v8i f;
  if constexpr (KC) {
    const int at = r0 * PITCH + kc_fragment<true, PITCH, false>(l, kstep);
    v4i lo = *US_LDS_PTR(const v4i, tile + at);
    v4i hi = *US_LDS_PTR(const v4i, tile + (at ^ 16));
    f = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
  } else {
    // 16 lanes cooperate on an 8(k) x 16(row) byte block: lane i points at k-row i/2, row-half i%2,
    // and receives the 8 k values of row (group base + i).  The swizzle only depends on k mod 8
    // (or (k/2) mod 4), which the four reads of a lane share.
    const int i = l & 15;
    const int krow = kstep * 64 + (l >> 5) * 32 + (i >> 1);
    const int col = r0 + ((l >> 4) & 1) * 16 + (i & 1) * 8;
    const uint32_t a = lds_addr(tile + krow * PITCH + (((col >> 4) ^ swz<false, true, PITCH, false>(krow)) << 4) + (col & 15));
    const v2i v0 = ds_read_tr8<0>(a), v1 = ds_read_tr8<8 * PITCH>(a), v2 = ds_read_tr8<16 * PITCH>(a),
              v3 = ds_read_tr8<24 * PITCH>(a);
    f = {v0.x, v0.y, v1.x, v1.y, v2.x, v2.y, v3.x, v3.y};
  }
  return f;
}

// (`index` of N fragments of a wave whose first row is r0.)  What depends on the lane is one value per operand and k-step.  Of a power of two of K-strided
// fragments, each 32 or 64 bytes wide, the first starts at a multiple of them all, and so do tiles and k-rows: the number of the fragment is a field of
// the LDS address.  (With an address of its own per fragment, a fifth more vector instructions per tile of a short reduction: us, before -> now, 4096 x 1024
// TN, K = 64 4.21 -> 4.10; 3072 x 1024 NT, K = 192 4.81 -> 4.67, K = 1024 10.8 -> 10.4; 16384 x 4096 NT, K = 64 29.7 -> 29.1.)
template <bool KC, int PITCH, int N, bool M16>
__device__ __forceinline__ v8h direct_frag_f16(const uint8_t* tile, int r0, int index, int kstep) {
  constexpr int ROWS = M16 ? 16 : 32;
  const int l = threadIdx.x & 63;
  if constexpr (KC) {
    const int at = (r0 + index * ROWS) * PITCH + kc_fragment<false, PITCH, M16>(l, kstep);
    return *US_LDS_PTR(const v8h, tile + at);
  } else {
    constexpr bool FIELD = (N & (N - 1)) == 0;
    uint32_t a = lds_addr(tile) + ks_fragment_f16<PITCH, M16>(l, FIELD ? r0 : r0 + index * ROWS, kstep);
    if constexpr (FIELD) a ^= (uint32_t)index * (2 * ROWS);
    const v2i lo = ds_read_tr16<0>(a), hi = ds_read_tr16<4 * PITCH>(a);
    v4i w = {lo.x, lo.y, hi.x, hi.y};
    v8h h;
    __builtin_memcpy(&h, &w, 16);
    return h;
  }
}

// FP8 fragments of the 16 x 16 x 128 instruction, 16 rows x 128 bytes of k: lane l supplies the 32 consecutive k of k-quarter l/16 of
// row l%16.  All reads are assembly, so that the main loop knows how many are pending; addresses are a register or two per operand and
// stage and constants (K-strided: one XOR per fragment, on the absolute address: DirectTile's assertions, the alignment of the kernels'
// dynamic LDS, and that there is no other LDS in front of it, which a test holds the built kernels to).
template <int OFFSET>
__device__ __forceinline__ v4i ds_read_16(uint32_t addr) {
  v4i v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFFSET));
  return v;
}
template <bool KC, int PITCH>
struct Frags128 {
  static constexpr int READS = KC ? 2 : 4;         // instructions per fragment
  uint32_t lane_off, at;
  // r0: the wave's first row of the tile, a multiple of 16 times the number of fragments; kstep: number of the 128 bytes of k
  __device__ __forceinline__ void init(int r0, int kstep) {
    const int l = threadIdx.x & 63;
    if constexpr (KC) {
      lane_off = (uint32_t)(r0 * PITCH + kc_fragment<true, PITCH, true>(l, kstep));
    } else {
      const int i = l & 15, krow = kstep * 128 + (l >> 4) * 32 + (i >> 1);
      lane_off = (uint32_t)(krow * PITCH + (((r0 >> 4) ^ swz<false, true, PITCH, true>(krow)) << 4) + (i & 1) * 8);
    }
  }
  __device__ __forceinline__ void open(uint32_t tile) { at = tile + lane_off; }
  template <int I>
  __device__ __forceinline__ v8i read() const {
    if constexpr (KC) {
      // (the second chunk: the swizzle's XOR and the chunk's own bit commute)
      const v4i lo = ds_read_16<I * 16 * PITCH>(at), hi = ds_read_16<I * 16 * PITCH>(at ^ 16u);
      return v8i{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    } else {
      const uint32_t a = at ^ (uint32_t)(I << 4);
      const v2i v0 = ds_read_tr8<0>(a), v1 = ds_read_tr8<8 * PITCH>(a), v2 = ds_read_tr8<16 * PITCH>(a), v3 = ds_read_tr8<24 * PITCH>(a);
      return v8i{v0.x, v0.y, v1.x, v1.y, v2.x, v2.y, v3.x, v3.y};
    }
  }
};
// Wait until at most N LDS reads are pending.  The counter has four bits: an operand of 15 is no wait at all, and what the counter does
// with a sixteenth pending read is not documented, so a wait that may leave more than 14 pending has to ask for 14.
constexpr int kMostCountedReads = 14;
template <int N>
__device__ __forceinline__ void lds_reads_pending() {
  static_assert(N >= 0 && N <= kMostCountedReads, "");
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}
template <int... I, class F>
__device__ __forceinline__ void static_for_each(std::integer_sequence<int, I...>, F f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
  static_for_each(std::make_integer_sequence<int, N>{}, f);
}

// A stage of RM x RN instructions with one set of fragments: the order of the instructions, and after how many of them each
// fragment of the next stage is requested.  The first two rows go column by column, the rest of the upper half of the rows row by row, the
// lower half column by column: so the fragments of the upper rows become free one after the other in the first half of the stage,
// those of the columns in the second half, and those of the lower rows are not needed until half of the next stage is over.
template <int RM, int RN>
struct KStep128 {
  static_assert(RM >= 4 && RM % 2 == 0 && RN >= 4, "");
  static constexpr int NMFMA = RM * RN, H = RM / 2, BOUNDARY = 2 * RN;
  // (one operand stays from each instruction to the next, but for one or two of them)
  static constexpr int row(int pos) {
    if (pos < BOUNDARY) return pos / 2 % 2 ? 1 - pos % 2 : pos % 2;
    if (pos < H * RN) return pos / RN;
    const int q = pos - H * RN;
    return H + (q / H % 2 ? H - 1 - q % H : q % H);
  }
  static constexpr int col(int pos) {
    if (pos < BOUNDARY) return pos / 2;
    if (pos < H * RN) return pos / RN % 2 ? RN - 1 - pos % RN : pos % RN;
    return (pos - H * RN) / H;
  }
  static constexpr int due_a(int i) {
    if (i == 0) return BOUNDARY;
    if (i == 1) return BOUNDARY + (H > 2 ? RN / 2 : 1);
    if (i < H) return (i + 1) * RN;
    return NMFMA + 1 + (i - H) * ((BOUNDARY - 4) / H);
  }
  static constexpr int due_b(int j) { return H * RN + (j + 1) * H; }
  // read instructions that may be pending ahead of instruction `pos` of the next stage (before the boundary) if fragment j of B is to
  // be there: those of the fragments requested behind it (NA, NB: instructions per fragment), as far as they can be counted
  template <int NA, int NB>
  static constexpr int pending_b(int j, int pos) {
    int n = 0;
    for (int k = j + 1; k < RN; ++k) n += NB;
    for (int i = H; i < RM; ++i) n += due_a(i) <= NMFMA + pos ? NA : 0;
    return n < kMostCountedReads ? n : kMostCountedReads;
  }
};

// s_waitcnt vmcnt(N) alone (lgkmcnt / expcnt fields left at "no wait")
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// One output tile (number `bid` in launch order, K slice `split`) by the whole workgroup; `lds` is the
// workgroup's dynamic LDS (DirectTile::LDS_BYTES).
template <class Cfg, bool FP8, int FA, int FB, bool A_KC, bool B_KC, int EPI, bool WIDE>
__device__ __forceinline__ void gemm_direct_tile(const GemmArgs& g, int bid, long split, uint8_t* lds) {
  using T = DirectTile<Cfg, FP8, A_KC, B_KC, WIDE, EPI>;
  constexpr int BM = Cfg::BM, BN = Cfg::BN, THREADS = Cfg::THREADS, BKB = Cfg::BKB, NST = Cfg::NST;
  constexpr int FM = Cfg::FM, FN = Cfg::FN;
  constexpr int ES = T::ES;
  constexpr int KSTEPS = BKB / (FP8 || T::M16 ? 64 : 32) / Cfg::WAVES_K;      // k-steps of a stage this wave works on
  using Acc = Accumulators<FM, FN, T::M16>;
  constexpr int RM = Acc::RM, RN = Acc::RN, RB = T::M16 ? 16 : 32;        // instruction results of the wave's tile, rows of one
  constexpr int PA = T::PA, PB = T::PB;
  constexpr int LOADS = T::A_LOADS + T::B_LOADS;       // per thread and stage

  int tm, tn;
  tile_of_block(g.walk, (uint32_t)bid, tm, tn);
  const long m0 = (long)tm * BM, n0 = (long)tn * BN;
  const long k_begin = split * g.k_per_split;
  const long k_end = (k_begin + g.k_per_split < g.K) ? k_begin + g.k_per_split : g.K;
  const int nstages = (k_end > k_begin) ? (int)((k_end - k_begin + T::BK - 1) / T::BK) : 0;
  const int krem = (int)((k_end - k_begin) - (long)(nstages - 1) * T::BK);       // elements of the last stage
  const bool ragged = krem != T::BK;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wmn = wave % Cfg::WAVES_MN;             // position in the output tile
  const int wk = wave / Cfg::WAVES_MN;              // share of the k-steps
  const int wm0 = (wmn % Cfg::WAVES_M) * Cfg::WM;
  const int wn0 = (wmn / Cfg::WAVES_M) * Cfg::WN;
  const int ks0 = wk * KSTEPS;

  OperandLoads<THREADS, BM, BKB, A_KC, FP8, PA, T::A_LOADS, T::M16> la;
  OperandLoads<THREADS, BN, BKB, B_KC, FP8, PB, T::B_LOADS, T::M16> lb;
  la.init(g.A, g.lda, m0, g.M, k_begin);
  lb.init(g.B, g.ldb, n0, g.N, k_begin);
  const long advA = A_KC ? (long)BKB : (long)T::BK * g.lda * ES;   // bytes per stage
  const long advB = B_KC ? (long)BKB : (long)T::BK * g.ldb * ES;

  Acc acc;
  acc.clear();

  auto load_number = [&](int l, __amdgpu_buffer_rsrc_t ra, __amdgpu_buffer_rsrc_t rb, uint8_t* stage_base) {
    if (l < T::A_LOADS) la.issue(l, ra, stage_base, wave);
    else lb.issue(l - T::A_LOADS, rb, stage_base + T::A_BYTES, wave);
  };
  auto next_stage = [&](__amdgpu_buffer_rsrc_t& ra, __amdgpu_buffer_rsrc_t& rb) {
    ra = la.resource();
    rb = lb.resource();
    la.next += advA;
    lb.next += advB;
  };
  // the resources of the next stage to request (number `stage`)
  auto open_stage = [&](int stage, __amdgpu_buffer_rsrc_t& ra, __amdgpu_buffer_rsrc_t& rb) {
    if (ragged && stage + 1 == nstages) {
      la.cut(krem);
      lb.cut(krem);
    }
    next_stage(ra, rb);
  };

  // The epilogue's second input (saved pre-activation / skip tensor): from the first boundary that refills
  // nothing any more, no wait of the main loop depends on the load counter, so one 4-byte load per 128-byte
  // line of this wave's share is sent off there (into the slot just freed, never read): the lines are in L2
  // when the epilogue asks for them instead of coming from HBM with every CU asking at once (BERT-large, backward
  // of layer 2: 97.4 -> 93.8 us, same box, same bits).
  auto prefetch_second_input = [&](int s, uint8_t* freed) {
    if constexpr (EPI == EPI_GELU_GRAD || EPI == EPI_GELU_GRAD_TAB || EPI == EPI_RESIDUAL) {
      if (s + NST == nstages) {
        constexpr int LPR = (Cfg::WN * 2 + 127) / 128;                 // lines per row of the wave's share
        constexpr int ROWS = Cfg::WM / Cfg::WAVES_K;                   // the rows this wave finishes
        const int lane = threadIdx.x & 63;
        uint8_t* dump = freed + wave * 256;
#pragma unroll
        for (int t = 0; t < ROWS * LPR; t += 64) {
          const int u = t + lane;
          const long m = m0 + wm0 + wk * ROWS + u / LPR;
          const long n = n0 + wn0 + (u % LPR) * 64;
          if (u < ROWS * LPR && m < g.M && n < g.N)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(g.Zpre + m * g.ldc + n),
                                             US_LDS_PTR(void, dump), 4, 0, 0);
        }
      }
    }
  };

  // prologue: fill the ring, open stage 0, fetch its first fragments
#pragma unroll
  for (int s = 0; s < NST; ++s)
    if (s < nstages) {
      __amdgpu_buffer_rsrc_t ra, rb;
      open_stage(s, ra, rb);
#pragma unroll
      for (int l = 0; l < LOADS; ++l) load_number(l, ra, rb, lds + s * T::STAGE_BYTES);
    }
  if (nstages > 0) {
    if (nstages >= NST) wait_vmcnt<(NST - 1) * LOADS>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
  }

  if constexpr (T::K128) {
    // FP8, one k-step of 128 bytes per stage and wave.  What bounds it on large products is power: next to the instruction of 32 x 32
    // results over 64 k, that of 16 x 16 over 128 moves its accumulators half as often (random data in registers, nothing else
    // running: 4.38 against 3.95 PFLOP/s; error against 64 bits the same over 4096 products).  (Not where the reduction has no more stages
    // than the ring: Short<Cfg>.)  Its fragments are twice as large per
    // k-step, so there is one set of them, and each is requested again behind its last instruction of the stage (KStep128).  The
    // stage boundary (own reads of stage s done, stage s+1 landed, barrier) lies behind the first two rows of results, and reads and
    // refills are spread over the stage: in bursts they hold the waves back (8192 x 8192, K = 8192 on zeros: 297 us like this, 336 with a
    // refill load per instruction, 344 with B's reads in the last two rows as well).
    // us, older form -> this, one box, random data: 8192 x 8192, K = 8192 NN 425 -> 409, NT 382 -> 360, TN 372 -> 357; 4096 x 4096, K = 4096 52.9 -> 50.8,
    // 53.4 -> 49.9, 55.1 -> 52.9; 32768 x 16384, K = 4096 NN 1826 -> 1750; the 32768 x 4096 x 16384 step 10.63 -> 10.19 ms.
    using Step = KStep128<RM, RN>;
    Frags128<A_KC, PA> ra128;
    Frags128<B_KC, PB> rb128;
    ra128.init(wm0, wk);
    rb128.init(wn0, wk);
    constexpr int NA = decltype(ra128)::READS, NB = decltype(rb128)::READS;
    v8i fa[RM], fb[RN];
    auto open_frags = [&](int slot) {
      const uint32_t stage = lds_addr(lds + slot * T::STAGE_BYTES);
      ra128.open(stage);
      rb128.open(stage + T::A_BYTES);
    };
    // the reads due once `done` instructions of a stage have been issued (NMFMA + x: x of the next one's)
    auto read_due = [&](auto done_) {
      constexpr int done = decltype(done_)::value;
      static_for<RM>([&](auto k) {
        if constexpr (Step::due_a(decltype(k)::value) == done) fa[decltype(k)::value] = ra128.template read<decltype(k)::value>();
      });
      static_for<RN>([&](auto k) {
        if constexpr (Step::due_b(decltype(k)::value) == done) fb[decltype(k)::value] = rb128.template read<decltype(k)::value>();
      });
    };
    // STEADY: the stage's slot is refilled; MORE: there is a next stage
    auto stage = [&](auto steady, auto more, int s, int slot) {
      constexpr bool STEADY = decltype(steady)::value, MORE = decltype(more)::value;
      __amdgpu_buffer_rsrc_t ra, rb;
      uint8_t* freed = lds + slot * T::STAGE_BYTES;
      static_for<Step::NMFMA>([&](auto pos_) {
        constexpr int pos = decltype(pos_)::value, i = Step::row(pos), j = Step::col(pos);
        if constexpr (pos < Step::BOUNDARY && pos % 2 == 0) {      // the first use of B's fragment j (and, at 0, of A's first rows)
          lds_reads_pending<Step::template pending_b<NA, NB>(j, pos)>();
          if constexpr (pos == 0) {
#pragma unroll
            for (int k = 0; k < RM / 2; ++k) asm volatile("" : "+v"(fa[k]));
          }
          asm volatile("" : "+v"(fb[j]));
        }
        acc.v[i][j] = mfma_fp8<FB, FA>(fb[j], fa[i], acc.v[i][j]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (pos + 1 < Step::BOUNDARY) read_due(std::integral_constant<int, Step::NMFMA + pos + 1>{});
        if constexpr (pos + 1 == Step::BOUNDARY) {
          lds_reads_done();
#pragma unroll
          for (int k = RM / 2; k < RM; ++k) asm volatile("" : "+v"(fa[k]));
          if constexpr (STEADY) {
            wait_vmcnt<(NST - 2) * LOADS>();   // stage s+1 has landed once only the NST-2 younger stages are pending
          } else if constexpr (MORE) {
            if (s + NST <= nstages) wait_vmcnt<(NST - 2) * LOADS>();
            else wait_vmcnt<0>();
          }
          __builtin_amdgcn_s_barrier();        // ... for everyone; nobody reads stage s any more
          if constexpr (STEADY) next_stage(ra, rb);
          else prefetch_second_input(s, freed);
          if constexpr (MORE) open_frags(slot + 1 == NST ? 0 : slot + 1);
        }
        if constexpr (MORE && pos + 1 >= Step::BOUNDARY) read_due(std::integral_constant<int, pos + 1>{});
        // the refill from the boundary on: spread over half of the stage, which keeps the vector-memory pipeline from holding a wave back
        // from the matrix core, or over a quarter of a short one, so that each load has most of a stage of time
        if constexpr (STEADY && pos >= Step::BOUNDARY) {
          constexpr int SPAN = Step::NMFMA >= 32 ? Step::NMFMA / 2 : Step::NMFMA / 4;
#pragma unroll
          for (int l = 0; l < LOADS; ++l)
            if (l * SPAN / LOADS == pos - Step::BOUNDARY) load_number(l, ra, rb, freed);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    if (nstages > 0) {
      open_frags(0);
      static_for<Step::NMFMA + 1>(read_due);
    }
    int slot = 0, s = 0;
    // The last stage is cut to what there is of the reduction between the passes of the outer loop: with a branch in its body the
    // compiler moves accumulators about where they take all accumulation registers (100 moves a stage of the four-wave tile).
    for (int uncut = ragged ? nstages - 1 : nstages;; uncut = nstages) {
      for (; s + NST < uncut; ++s) {
        stage(std::true_type{}, std::true_type{}, s, slot);
        if (++slot == NST) slot = 0;
      }
      if (uncut == nstages) break;
      la.cut(krem);
      lb.cut(krem);
    }
    for (; s + 1 < nstages; ++s) {
      stage(std::false_type{}, std::true_type{}, s, slot);
      if (++slot == NST) slot = 0;
    }
    if (s < nstages) stage(std::false_type{}, std::false_type{}, s, slot);
  } else {
    // fragment registers, two sets: one feeds the MFMAs while the other is being filled
    using FragT = typename std::conditional<FP8, v8i, v8h>::type;
    FragT fa[2][RM], fb[2][RN];
    auto load_frags = [&](FragT (&a)[RM], FragT (&b)[RN], int slot, int ks) {
      const uint8_t* ta = lds + slot * T::STAGE_BYTES;
      const uint8_t* tb = ta + T::A_BYTES;
#pragma unroll
      for (int j = 0; j < RN; ++j) {
        if constexpr (FP8) b[j] = direct_frag_fp8<B_KC, PB>(tb, wn0 + j * RB, ks0 + ks);
        else b[j] = direct_frag_f16<B_KC, PB, RN, T::M16>(tb, wn0, j, ks0 + ks);
      }
#pragma unroll
      for (int i = 0; i < RM; ++i) {
        if constexpr (FP8) a[i] = direct_frag_fp8<A_KC, PA>(ta, wm0 + i * RB, ks0 + ks);
        else a[i] = direct_frag_f16<A_KC, PA, RM, T::M16>(ta, wm0, i, ks0 + ks);
      }
    };
    // one fragment of a k-step: numbers 0 .. RN-1 are the B fragments, RN .. RN+RM-1 the A fragments
    auto load_frag_one = [&](FragT (&a)[RM], FragT (&b)[RN], int slot, int ks, int idx) {
      const uint8_t* ta = lds + slot * T::STAGE_BYTES;
      const uint8_t* tb = ta + T::A_BYTES;
      if (idx < RN) {
        if constexpr (FP8) b[idx] = direct_frag_fp8<B_KC, PB>(tb, wn0 + idx * RB, ks0 + ks);
        else b[idx] = direct_frag_f16<B_KC, PB, RN, T::M16>(tb, wn0, idx, ks0 + ks);
      } else {
        const int i = idx - RN;
        if constexpr (FP8) a[i] = direct_frag_fp8<A_KC, PA>(ta, wm0 + i * RB, ks0 + ks);
        else a[i] = direct_frag_f16<A_KC, PA, RM, T::M16>(ta, wm0, i, ks0 + ks);
      }
    };
    if (nstages > 0) load_frags(fa[0], fb[0], 0, 0);

    // The two fragment sets alternate per k-step.  With an odd number of k-steps per stage (one) the
    // loop body therefore spans two stages, so that the set index stays a compile-time constant.
    constexpr int SPI = (KSTEPS % 2) ? 2 : 1;     // stages per loop iteration
    int slot = 0;                                 // ring slot of the current stage
    // STEADY: every stage of the iteration is followed by one more and its slot is refilled; otherwise the end of the loop
    auto iteration = [&](auto steady, int s0) {
      constexpr bool STEADY = decltype(steady)::value;
      __amdgpu_buffer_rsrc_t ra, rb;
#pragma unroll
      for (int u = 0; u < SPI * KSTEPS; ++u) {
        const int s = s0 + u / KSTEPS;
        const int ks = u % KSTEPS;
        if (!STEADY && SPI > 1 && s >= nstages) break;       // odd stage count: the last iteration is half empty
        FragT (&ca)[RM] = fa[u & 1];
        FragT (&cb)[RN] = fb[u & 1];
        FragT (&na)[RM] = fa[(u + 1) & 1];
        FragT (&nb)[RN] = fb[(u + 1) & 1];
        // the fragments of this k-step were requested one k-step ago
        lds_reads_done();
        frag_ready(ca);
        frag_ready(cb);
        // The next k-step's fragments are not requested ahead of this k-step's MFMAs but one at a time behind the later ones,
        // so that a wave that comes out of a wait (or the barrier) feeds the matrix core first.  FP8, behind the last FM + FN of them
        // (measured when the 256 x 256 tile ran this loop as well: 2.47 -> 2.64 PFLOP/s on a 32768 x 4096 x 16384 product, BERT-large step 256 -> 247 us;
        // behind the first MFMAs instead: 2.55; two per MFMA behind the last three: 2.57; all behind the last: 2.50).
        // FP16, instructions of 32 x 32 results: few tiles' or narrow ones', whose stages are short, ahead of them; of 16 x 16, evenly from a quarter of them on (us, ahead of all / evenly from the first / from a quarter on, refills below over all of
        // them: 8192 x 8192, K = 8192 NN 848 / 814 / 793, 4096 x 768, K = 3072 NN on W128 25.2 / 23.7 / 23.2).
        const bool boundary = ks + 1 == KSTEPS;
        const bool more = STEADY || !boundary || s + 1 < nstages;     // there is a next k-step
        bool refill = false;
        uint8_t* refill_base = lds + slot * T::STAGE_BYTES;
        if (boundary) {
          // stage boundary: this wave holds all of stage s in registers
          if constexpr (STEADY) {
            wait_vmcnt<(NST - 2) * LOADS>();     // own loads of stage s+1 have landed once only the NST-2 younger stages are pending
          } else if (s + 1 < nstages) {
            if (s + NST <= nstages) wait_vmcnt<(NST - 2) * LOADS>();
            else wait_vmcnt<0>();
          }
          __builtin_amdgcn_s_barrier();   // stage s+1 complete for everyone; nobody reads stage s any more
          // the freed slot receives stage s+NST, a few loads per MFMA below
          refill = STEADY || (SPI > 1 && s + NST < nstages);
          if (refill) open_stage(s + NST, ra, rb);
          if constexpr (!STEADY) prefetch_second_input(s, refill_base);
          if (++slot == NST) slot = 0;
        }
        const int fks = boundary ? 0 : ks + 1;
        constexpr bool AHEAD = !FP8 && !T::M16;
        if constexpr (AHEAD) {
          if (more) load_frags(na, nb, slot, fks);
        }
        __builtin_amdgcn_sched_barrier(0);
        // The refill loads are spread over the MFMAs of this k-step: issued in one burst by all waves
        // they would queue up in the vector-memory pipeline and hold the waves back from the matrix core.
        constexpr int NMFMA = RM * RN;
#pragma unroll
        for (int i = 0; i < RM; ++i)
#pragma unroll
          for (int jj = 0; jj < RN; ++jj) {
            const int j = T::M16 && (i & 1) ? RN - 1 - jj : jj;      // 16 x 16: one operand stays from each instruction to the next
            if constexpr (FP8) acc.v[i][j] = mfma_fp8<FB, FA>(cb[j], ca[i], acc.v[i][j]);
            else acc.v[i][j] = mfma_f16(cb[j], ca[i], acc.v[i][j]);
            const int pos = i * RN + jj;
            constexpr int NFR = RM + RN;
            constexpr int FIRST = FP8 ? (NMFMA > NFR ? NMFMA - NFR : 0) : NMFMA / 4;
#pragma unroll
            for (int idx = 0; idx < NFR; ++idx)
              if (!AHEAD && FIRST + idx * (NMFMA - FIRST) / NFR == pos && more) load_frag_one(na, nb, slot, fks, idx);
            __builtin_amdgcn_sched_barrier(0);
            if (boundary) {
              constexpr int SPAN = FP8 && LOADS < NMFMA ? LOADS : NMFMA;
#pragma unroll
              for (int l = 0; l < LOADS; ++l)
                if (l * SPAN / LOADS == pos && refill) load_number(l, ra, rb, refill_base);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        __builtin_amdgcn_sched_barrier(0);   // ... and the MFMAs ahead of the next k-step's wait
      }
    };
    int s0 = 0;
    for (; s0 + SPI - 1 + NST < nstages; s0 += SPI) iteration(std::true_type{}, s0);
    for (; s0 < nstages; s0 += SPI) iteration(std::false_type{}, s0);
  }

  __syncthreads();       // every wave is past its last fragment read before the strips overlay the ring
  if constexpr (Cfg::WAVES_K > 1) {
    // Two wave groups hold partial sums of the same tile.  Each group finishes one half of the rows:
    // it hands the other half of its accumulators to its partner through LDS and adds the partner's
    // half to its own (one addition of two terms per element, so the order does not matter and the
    // result is deterministic).  Quad q of lane l travels through red[wk][wmn][q][l].
    static_assert(Cfg::WAVES_K == 2 && FM % 2 == 0, "two groups, an even number of 32-row blocks");
    constexpr int HALF = FM / 2, NQ = HALF * FN * 4;
    v4f* red = reinterpret_cast<v4f*>(lds);
    const int lane = threadIdx.x & 63;
    v4f* mine = red + ((size_t)(wk * Cfg::WAVES_MN + wmn) * NQ) * 64 + lane;
    const v4f* theirs = red + ((size_t)((wk ^ 1) * Cfg::WAVES_MN + wmn) * NQ) * 64 + lane;
    auto send = [&](auto I0c) {          // the rows the partner finishes
      constexpr int I0 = decltype(I0c)::value;
#pragma unroll
      for (int i = 0; i < HALF; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) *US_LDS_PTR(v4f, mine + ((i * FN + j) * 4 + q) * 64) = acc.quad(I0 + i, j, q);
    };
    auto receive = [&](auto I0c) {       // the rows this wave finishes
      constexpr int I0 = decltype(I0c)::value;
#pragma unroll
      for (int i = 0; i < HALF; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
#pragma unroll
          for (int q = 0; q < 4; ++q) acc.add(I0 + i, j, q, *US_LDS_PTR(const v4f, theirs + ((i * FN + j) * 4 + q) * 64));
          __builtin_amdgcn_sched_barrier(0);   // one block of 16 at a time keeps the register count down
        }
    };
    if (wk == 0) send(std::integral_constant<int, HALF>{});
    else send(std::integral_constant<int, 0>{});
    __syncthreads();
    if (wk == 0) receive(std::integral_constant<int, 0>{});
    else receive(std::integral_constant<int, HALF>{});
    __syncthreads();     // everything exchanged: the strips may overlay the exchange area
    if (wk == 0) store_block_epilogue<Cfg, EPI, WIDE, 0, HALF, epilogue_takes_bias<A_KC, B_KC, EPI, WIDE>()>(g, acc, lds, m0, n0, split);
    else store_block_epilogue<Cfg, EPI, WIDE, HALF, FM, epilogue_takes_bias<A_KC, B_KC, EPI, WIDE>()>(g, acc, lds, m0, n0, split);
    return;
  }
  store_block_epilogue<Cfg, EPI, WIDE, 0, Cfg::FM, epilogue_takes_bias<A_KC, B_KC, EPI, WIDE>()>(g, acc, lds, m0, n0, split);
}

template <class Cfg, bool FP8, int FA, int FB, bool A_KC, bool B_KC, int EPI, bool WIDE>
__global__ void __launch_bounds__(Cfg::THREADS, Cfg::MINB) gemm_direct_kernel(GemmArgs g) {
  extern __shared__ __attribute__((aligned(256))) uint8_t lds[];
  if constexpr (EPI == EPI_STORE) select_batch_item(g);
  gemm_direct_tile<Cfg, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(g, (int)blockIdx.x, (long)blockIdx.y, lds);
}

// Two batches of equally shaped products in one launch (attention's dV and dK: P^T dO and dA^T Q per head): one start-up and one
// drain instead of two.  All tiles of an item go to one XCD, whose L2 then serves the narrow operand to all of them.
struct BatchWalk {
  FastDiv by_xcds, by_tiles;
  uint32_t xcds, tiles;      // tiles of an item
  int batch;
};
template <class Cfg, bool FP8, int FA, int FB, bool A_KC, bool B_KC>
__global__ void __launch_bounds__(Cfg::THREADS, Cfg::MINB) gemm_two_batches_kernel(BatchWalk w, GemmArgs a, GemmArgs b) {
  extern __shared__ __attribute__((aligned(256))) uint8_t lds[];
  const uint32_t i = w.by_xcds.of(blockIdx.x), xcd = blockIdx.x - i * w.xcds, row = w.by_tiles.of(i);
  const int item = (int)(row * w.xcds + xcd), tile = (int)(i - row * w.tiles);
  if (item >= 2 * w.batch) return;
  GemmArgs g = item < w.batch ? a : b;
  const long z = item < w.batch ? item : item - w.batch;
  g.A += z * g.batch_a;
  g.B += z * g.batch_b;
  g.C = (uint8_t*)g.C + z * g.batch_c;
  gemm_direct_tile<Cfg, FP8, FA, FB, A_KC, B_KC, EPI_STORE, false>(g, tile, 0, lds);
}

// Two independent GEMMs in one launch (the two products of a layer's backward pass), for tile shapes
// with the same workgroup size: the first nb workgroups work on problem B (grad_W: few tiles, long main
// loop), the rest on problem A (grad_X).  Compared with two launches there is no drain between the
// two, and because the B tiles finish at slightly different times the A tiles start staggered: their
// epilogues (GELU' over a large output: a burst of HBM reads, vector ALU work, HBM writes) no longer
// hit every CU at the same moment, while launched on their own all CUs run in lockstep.  (Interleaving
// A and B tiles more finely was measured to be slower than either.)
// (The A tiles count from the first workgroup behind the B tiles: another nb only renames the XCDs of their walk.)
template <class Cfg, bool FP8, int FA, int FB, bool A_KC, bool B_KC, int EPI, bool WIDE>
struct GemmKind {
  using Tile = DirectTile<Cfg, FP8, A_KC, B_KC, WIDE, EPI>;
  static constexpr int THREADS = Cfg::THREADS, BM = Cfg::BM, BN = Cfg::BN, MINB = Cfg::MINB;
  static constexpr int WAVES_K = Cfg::WAVES_K, NST = Cfg::NST, EPI_ = EPI;
  static constexpr bool IS_FP8 = FP8, A_KC_ = A_KC, B_KC_ = B_KC;
  __device__ static __forceinline__ void run(const GemmArgs& g, int bid, uint8_t* lds) {
    gemm_direct_tile<Cfg, FP8, FA, FB, A_KC, B_KC, EPI, WIDE>(g, bid, 0, lds);
  }
};

template <class KA, class KB>
__global__ void __launch_bounds__(KA::THREADS, KA::MINB < KB::MINB ? KA::MINB : KB::MINB) gemm_pair_kernel(int nb, GemmArgs a, GemmArgs b) {
  static_assert(KA::THREADS == KB::THREADS, "one workgroup size for both problems");
  extern __shared__ __attribute__((aligned(256))) uint8_t lds[];
  const int bid = (int)blockIdx.x;
  if (bid < nb) KB::run(b, bid, lds);
  else KA::run(a, bid - nb, lds);
}

}  // namespace us
