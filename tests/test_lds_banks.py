"""The LDS swizzle of K-contiguous operand tiles (us::swz, us::kc_fragment), compiled for the host: the 16 lanes that a 16-byte LDS read serves together
meet every group of four banks once, for each fragment form but FP16's of 16 rows at a pitch of 64 bytes; the chunks of a row stay in the row, each in a place of its own; and
a row 16 further down has the same mask, which the constant offsets between the fragments of a wave rely on.  Of K-strided FP16 tiles (us::ks_fragment_f16): the
32 lanes served together meet no bank twice, and a fragment's number is a field of the address where a wave has a power of two of them."""
import subprocess

from paper_2303_11257_amd import build

SOURCE = """
#include "us_gemm_direct.h"
#include <cstdio>
using namespace us;

template <bool FP8, int PITCH, bool M16>
static int check() {
  static const int served[2][16] = {{0, 1, 2, 3, 12, 13, 14, 15, 20, 21, 22, 23, 24, 25, 26, 27}, {4, 5, 6, 7, 8, 9, 10, 11, 16, 17, 18, 19, 28, 29, 30, 31}};
  for (int row = 0; row < 256; ++row) {
    unsigned seen = 0;
    for (int chunk = 0; chunk < PITCH / 16; ++chunk) seen |= 1u << (chunk ^ swz<true, FP8, PITCH, M16>(row));
    if (seen != (1u << PITCH / 16) - 1 || swz<true, FP8, PITCH, M16>(row) != swz<true, FP8, PITCH, M16>(row + 16)) return printf("mask of row %d\\n", row);
  }
  for (int kstep = 0; kstep < PITCH / 64 / (FP8 && M16 ? 2 : 1); ++kstep)
    for (int flip = 0; flip <= (FP8 ? 16 : 0); flip += 16)
      for (int phase = 0; phase < 4; ++phase) {
        unsigned banks = 0;
        for (int k = 0; k < 16; ++k)
          banks |= 1u << ((kc_fragment<FP8, PITCH, M16>(served[phase % 2][k] + phase / 2 * 32, kstep) ^ flip) / 16 % 16);
        if (banks != 0xffff) return printf("FP8 %d, pitch %d, 16 x 16 %d: k-step %d, phase %d: %x\\n", FP8, PITCH, M16, kstep, phase, banks);
      }
  return 0;
}

template <int PITCH, bool M16>
static int check_strided() {
  for (int kstep = 0; kstep < 2; ++kstep)
    for (int half = 0; half < 64; half += 32) {
      unsigned banks = 0;                          // pairs of banks: eight bytes per lane
      for (int l = half; l < half + 32; ++l) banks |= 1u << ks_fragment_f16<PITCH, M16>(l, 0, kstep) / 8 % 32;
      if (banks != 0xffffffff) return printf("K-strided, pitch %d, k-step %d, lanes from %d: %x\\n", PITCH, kstep, half, banks);
    }
  const int rows = M16 ? 16 : 32;
  for (int n = 1; n <= 128 / rows && 2 * rows * n <= PITCH; n *= 2)
    for (int base = 0; base < 1024; base += 256)
      for (int r0 = 0; 2 * r0 < PITCH; r0 += rows * n)
        for (int index = 0; index < n && PITCH % (2 * rows * n) == 0; ++index)
          for (int l = 0; l < 64; ++l)
            if (((base + ks_fragment_f16<PITCH, M16>(l, r0, 1)) ^ index * 2 * rows) != base + ks_fragment_f16<PITCH, M16>(l, r0 + rows * index, 1))
              return printf("pitch %d, fragment %d of %d from row %d\\n", PITCH, index, n, r0);
  return 0;
}

int main() {
  if (check_strided<64, true>() || check_strided<128, true>() || check_strided<256, true>() || check_strided<384, true>() || check_strided<512, true>()) return 1;
  if (check_strided<64, false>() || check_strided<128, false>() || check_strided<256, false>() || check_strided<384, false>() || check_strided<512, false>()) return 1;
  if (check<true, 128, true>() || check<true, 128, false>() || check<true, 64, false>() || check<false, 128, true>() || check<false, 128, false>() || check<false, 64, false>()) return 1;
  printf("ok\\n");
}
"""


def test_k_contiguous_fragments_meet_no_bank_twice(tmp_path):
    src, exe = tmp_path / "banks.hip", tmp_path / "banks"
    src.write_text(SOURCE)
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, "--offload-host-only", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.stdout == "ok\n", r.stdout + r.stderr
