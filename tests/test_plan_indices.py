"""Index arithmetic of the plan kernel at sizes no test can run at: the header's host / device functions
compiled for the host."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "epd_internal.h"
#include <cstdio>
using namespace epd;
// Walks the blocks around `first` and the last ones of a table of T x pairs entries: every entry once, in
// order, at its own place, nothing beyond the table.
static bool walk(int T, int pairs, int from_token, int to_token) {
  const int tpb = rot_tokens_per_block(pairs);
  int tok = from_token / tpb * tpb, pair = 0;
  for (int b = from_token / tpb; b <= (to_token - 1) / tpb; ++b)
    for (int t = 0; t < 256; ++t) {
      RotEntry e;
      if (!rot_entry(T, pairs, b, t, e)) continue;
      if (e.tok != tok || e.pair != pair || e.at != (unsigned long long)tok * pairs + pair || e.tok >= T) {
        std::printf("T %d pairs %d block %d thread %d: token %d pair %d at %zu, not token %d pair %d\n", T, pairs, b, t, e.tok, e.pair, e.at, tok, pair);
        return false;
      }
      if (++pair == pairs) { pair = 0; ++tok; }
    }
  return pair == 0 && tok >= to_token;
}
int main() {
  for (int pairs : {1, 4, 5, 16, 32, 36, 40, 48, 64})
    for (int T : {1, 7, 256, 100003, 1 << 26, (1 << 30) - 200}) {
      const int mid = (int)((1ll << 31) / pairs);                       // where 31 bits end
      if (!walk(T, pairs, 0, T < 600 ? T : 600) || !walk(T, pairs, T > 600 ? T - 600 : 0, T)) return 1;
      if (mid > 300 && mid + 300 < T && !walk(T, pairs, mid - 300, mid + 300)) return 1;
    }
  std::puts("walked");
}
"""


@pytest.mark.skipif(not os.path.isdir("/opt/rocm/include/hip"), reason="no HIP headers")
def test_rotary_entries_are_each_made_once_at_their_own_place(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2601_11590_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=120)
    assert r.returncode == 0 and "walked" in r.stdout, r.stdout
