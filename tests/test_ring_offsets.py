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
      const unsigned got = ring_sub_tile(t, bk, end, K, rb);
      if (t < kb + nk ? got != (unsigned)(t * bk) * rb : got < (unsigned)K * rb) {{ std::printf("range %d, sub-tile %d: %u\\n", sp, t, got); return 1; }}
    }}
  }}
""")


@pytest.mark.parametrize("bk,sz", [(32, 2), (64, 2), (128, 2), (64, 4)])
def test_no_k_row_past_the_sum_comes_round_to_one_that_is_there(tmp_path, bk, sz):
    """Every load that a ring issues, up to four sub-tiles past the last one, of operands from packed to the widest that it takes: rows of the sum
    are read where they lie, the others past the operand."""
    _program(tmp_path, f"""
  const int bk = {bk}, sz = {sz};
  const int Ks[] = {{1, 2, 5, 13, bk - 1, bk, bk + 1, 3 * bk - 1, 4 * bk + 7, 1000}};
  for (int K : Ks) {{
    const long most = (0x7ffff000L - 1) / sz / K / 8 * 8;  // the largest ld, in chunks
    const long lds[] = {{8, 264, 4090440, 4090448, 17200000, 34500000, 70000000, 140000000, most / 2 / 8 * 8, most - 8, most}};
    if (!ring_spans(K, most, sz) || ring_spans(K, most + 8, sz)) return 2;
    for (long ld : lds) {{
      if (ld < 8 || !ring_spans(K, ld, sz)) continue;
      const unsigned rb = (unsigned)(ld * sz);
      const int nk = (K + bk - 1) / bk;
      for (int t = 0; t < nk + 4; ++t)
        for (int k = 0; k < bk; ++k)
          for (unsigned col = 0; col < 2048; col += 496) {{
            const unsigned got = ring_lane(k, K, rb, col) + ring_sub_tile(t, bk, K, K, rb);
            const long row = (long)t * bk + k;
            if (row < K ? got != row * (long)rb + col : got < (unsigned long)K * rb) {{
              std::printf("K %d, ld %ld, row %ld, column byte %u: %u\\n", K, ld, row, col, got);
              return 1;
            }}
          }}
    }}
  }}
""")


def test_columns_of_a_wider_matrix_are_not_read_behind_it(tmp_path):
    """An operand that is the last columns of a matrix: what a descriptor spans holds all of the operand's chunks and ends inside the matrix, whose
    rows a product wants to be whole chunks."""
    _program(tmp_path, """
  for (long sz : {2L, 4L})
    for (long K : {1L, 7L, 4096L})
      for (long n : {1L, 8L, 60L, 200L, 320L, 768L})
        for (long first : {0L, 8L, 640L, 1536L}) {
          const long e = 16 / sz, ld = (first + n + e - 1) / e * e, at = first * sz, got = k_slow_bytes(K, ld, n, sz);
          if (at + got > K * ld * sz || got < ((K - 1) * ld + n) * sz || got % 16) { std::printf("%ld %ld %ld %ld: %ld\\n", sz, K, n, first, got); return 1; }
        }
""")
