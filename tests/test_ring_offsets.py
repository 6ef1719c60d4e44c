"""Offsets of the direct-to-LDS ring's loads of an operand with k as the slow index (csrc/ring_offsets.h) against plain arithmetic in 64 bits: what
is inside the sum is read where it lies, and nothing else is fetched.  Host code without HIP: a small program around it runs on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _program(tmp_path, body):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <algorithm>\n#include <cstdio>\n#include "ring_offsets.h"\nusing namespace hydra;\nint main() {\n' + body + "}\n")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2107_06469_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("K,S", [(2048, 2), (2080, 2), (8192, 8), (9000, 7), (3104, 3)])
def test_a_range_of_a_split_sum_fetches_nothing_of_the_next_one(tmp_path, K, S):
    """Ranges as gemm_dma_kernel divides them (sub-tiles of 32 k); a ring of four stages asks for three sub-tiles past the range's last."""
    _program(tmp_path, f"""
  const int K = {K}, S = {S}, bk = 32, nk_all = (K + bk - 1) / bk, per = (nk_all + S - 1) / S;
  const unsigned rb = 2 * 776;
  for (int sp = 0; sp < S; ++sp) {{
    const int kb = sp * per, nk = std::max(0, std::min(nk_all, kb + per) - kb), end = std::min(K, (kb + nk) * bk);
    for (int t = kb; t < kb + nk + 3; ++t) {{
      const unsigned got = ring_sub_tile(t, bk, end, rb);
      if (t < kb + nk ? got != (unsigned)(t * bk) * rb : got < (unsigned)K * rb) {{ std::printf("range %d, sub-tile %d: %u\\n", sp, t, got); return 1; }}
    }}
  }}
""")
