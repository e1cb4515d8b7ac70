"""The order of a stage's matrix instructions and fragment reads in the FP8 main loop (us::KStep128), pure constants, compiled for the host and played over
several stages, with the waits where the kernel has them: every result once per stage, every operand the one of its stage, no fragment requested again
before its last use, and the counted LDS waits long enough.  (Ring slots, their refills and the counted waits for those are not part of this: the tests of
ragged reductions run them on the device.)"""
import subprocess

from paper_2303_11257_amd import build

SOURCE = """
#include "us_gemm_direct.h"
#include <cstdio>
#include <vector>
using namespace us;

template <int RM, int RN, int NA, int NB>
static int play() {
  using S = KStep128<RM, RN>;
  std::vector<int> a(RM, -1), b(RN, -1);         // the stage a fragment's registers hold or will hold
  std::vector<int> order;                        // fragments in the order they were requested (A: 0 .., B: RM ..)
  std::vector<int> done(RM + RN, -1);            // the stage whose fragment is known to have arrived
  auto request = [&](int due, int stage) {
    for (int i = 0; i < RM; ++i)
      if (S::due_a(i) == due) { a[i] = stage; order.push_back(i); }
    for (int j = 0; j < RN; ++j)
      if (S::due_b(j) == due) { b[j] = stage; order.push_back(RM + j); }
  };
  auto wait = [&](int instructions) {            // all but the last `instructions` reads have arrived
    int pending = 0;
    for (int k = (int)order.size() - 1; k >= 0; --k) {
      pending += order[k] < RM ? NA : NB;
      if (pending > instructions) done[order[k]] = order[k] < RM ? a[order[k]] : b[order[k] - RM];
    }
  };
  for (int i = 0; i < RM; ++i)
    if (S::due_a(i) < S::BOUNDARY || S::due_a(i) >= S::NMFMA + S::BOUNDARY) return printf("due a %d\\n", i);
  for (int j = 0; j < RN; ++j)
    if (S::due_b(j) < S::BOUNDARY || S::due_b(j) > S::NMFMA) return printf("due b %d\\n", j);
  for (int due = 0; due <= S::NMFMA; ++due) request(due, 0);
  for (int s = 0; s < 4; ++s) {
    std::vector<int> seen(RM * RN, 0);
    for (int pos = 0; pos < S::NMFMA; ++pos) {
      const int i = S::row(pos), j = S::col(pos);
      if (i < 0 || i >= RM || j < 0 || j >= RN || seen[i * RN + j]++) return printf("result %d %d at %d\\n", i, j, pos);
      if (pos < S::BOUNDARY && pos % 2 == 0) {
        const int n = S::template pending_b<NA, NB>(j, pos);
        if (n < 15) wait(n);                     // the counter has four bits: with an operand of 15 the instruction waits for nothing
      }
      if (a[i] != s || b[j] != s || done[i] != s || done[RM + j] != s) return printf("operands of %d %d at %d, stage %d\\n", i, j, pos, s);
      if (pos + 1 < S::BOUNDARY) request(S::NMFMA + pos + 1, s);
      if (pos + 1 == S::BOUNDARY) {
        wait(0);
        for (int k : a) if (k != s) return printf("A not read at the boundary\\n");
        for (int k : b) if (k != s) return printf("B not read at the boundary\\n");
        order.clear();
      }
      if (pos + 1 >= S::BOUNDARY) request(pos + 1, s + 1);
    }
  }
  return 0;
}

int main() {
  if (play<8, 8, 2, 2>() || play<8, 8, 2, 4>() || play<8, 8, 4, 4>() || play<8, 4, 2, 2>() || play<8, 4, 2, 4>() || play<8, 4, 4, 4>() ||
      play<4, 4, 2, 2>() || play<4, 4, 2, 4>() || play<4, 4, 4, 4>())
    return 1;
  printf("ok\\n");
}
"""


def test_stage_schedule(tmp_path):
    src, exe = tmp_path / "stage.hip", tmp_path / "stage"
    src.write_text(SOURCE)
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, "--offload-host-only", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.stdout == "ok\n", r.stdout + r.stderr
