"""The host's part of the walk over a matmul's tiles, pure integer arithmetic, compiled for the host: division by a prepared divisor against the
machine's, and the place of every workgroup against the walk written with plain divisions; every tile exactly once."""
import subprocess

from paper_2303_11257_amd import build

SOURCE = """
#include "us_gemm_common.h"
#include <cstdio>
#include <vector>
using namespace us;

static int fail(const char* what, long a, long b, long c) { printf("%s %ld %ld %ld\\n", what, a, b, c); return 1; }

// XCD x of the workgroup id gets a rectangle of rm x rn tiles, walked in bands of 8 columns, columns fastest
static void plain(int bid, int tiles_m, int tiles_n, int gm, int gn, int nxcd, int& tm, int& tn) {
  int rm = tiles_m, rn = tiles_n, base_m = 0, base_n = 0, idx = bid;
  if (gm != 0) {
    rm = tiles_m / gm;
    rn = tiles_n / gn;
    base_m = bid % nxcd % gm * rm;
    base_n = bid % nxcd / gm * rn;
    idx = bid / nxcd;
  }
  const int band = idx / (rm * 8), r = idx - band * rm * 8, w = rn - band * 8 < 8 ? rn - band * 8 : 8;
  tm = base_m + r / w;
  tn = base_n + band * 8 + r % w;
}

static int grid(int m, int n, int nxcd) {
  int gm, gn;
  choose_xcd_grid(m, n, nxcd, 128, 128, gm, gn);
  const TileWalk walk(m, n, nxcd, gm, gn, 8);
  std::vector<char> seen(m * n);
  for (int bid = 0; bid < m * n; ++bid) {
    int tm, tn, pm, pn;
    tile_of_block(walk, bid, tm, tn);
    plain(bid, m, n, gm, gn, nxcd, pm, pn);
    if (tm != pm || tn != pn) return fail("tile", m, n, bid);
    if (tm < 0 || tm >= m || tn < 0 || tn >= n || seen[tm * n + tn]++) return fail("twice", m, n, bid);
  }
  return 0;
}

int main() {
  std::vector<uint32_t> values;
  for (uint32_t v = 0; v < 300; ++v) values.push_back(v);
  for (int s = 8; s < 32; ++s)
    for (int o = -3; o <= 3; ++o) values.push_back((1u << s) + o);
  for (uint32_t v = 1000003u; v < 4000000000u; v += 62345679u) values.push_back(v);
  for (int o = 1; o < 4; ++o) values.push_back(0u - o);
  for (uint32_t d : values) {
    if (d < 1 || d >= (1u << 31)) continue;
    const FastDiv by = FastDiv::by(d);
    for (uint32_t n : values)
      if (by.of(n) != n / d || by.of(n * d) != n * d / d) return fail("division", n, d, by.of(n));
  }
  for (int m = 1; m <= 48; ++m)
    for (int n = 1; n <= 48; ++n)
      for (int nxcd : {1, 2, 6, 8})
        if (grid(m, n, nxcd)) return 1;
  const int wide[][2] = {{1, 30000}, {30000, 1}, {8, 9000}, {9000, 8}, {1000, 77}, {77, 1000}, {512, 512}};
  for (auto& s : wide)
    if (grid(s[0], s[1], 8)) return 1;
  printf("ok\\n");
}
"""


def test_tile_walk(tmp_path):
    src, exe = tmp_path / "walk.hip", tmp_path / "walk"
    src.write_text(SOURCE)
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, "--offload-host-only", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.stdout == "ok\n", r.stdout + r.stderr
