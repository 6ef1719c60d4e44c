"""The rules that choose a tile for large launches (csrc/gemm_rules.h) at counts where both tiles were measured: what was slower is not chosen.
The rules are host code without HIP: a small program around them runs on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _chosen(tmp_path, calls):
    """Values of the calls, expressions in C++."""
    if not shutil.which("g++"):
        pytest.skip("no g++")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cstdio>\n#include "gemm_rules.h"\nusing namespace hydra;\nint main() {\n'
                   + "".join(f'  std::printf("%d\\n", (int)({c}));\n' for c in calls) + "}\n")
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2107_06469_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    return [int(x) for x in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]


def test_products_with_a_thin_last_pass(tmp_path):
    # (256x256 tiles, 128x128 tiles, K, gate or pre-activation, 128x128 tiles are ahead)
    cases = [(288, 1152, 768, 1, 1), (288, 1152, 3072, 1, 1), (320, 1280, 3072, 1, 1), (384, 1536, 768, 0, 1), (384, 1536, 3072, 0, 1),
             (377, 1450, 3072, 0, 1), (576, 2304, 3072, 0, 1), (640, 2560, 768, 0, 1), (640, 2560, 768, 1, 1), (832, 3328, 768, 0, 1),
             (800, 3200, 512, 1, 1), (860, 3440, 768, 1, 1), (1050, 4200, 768, 1, 1), (400, 1600, 512, 1, 1), (414, 1656, 256, 1, 1),
             # a fourth 128x128 tile to a pass: behind
             (390, 1560, 768, 0, 0), (390, 1560, 3072, 0, 0), (390, 1560, 3072, 1, 0), (390, 1560, 1024, 0, 0), (400, 1600, 768, 0, 0),
             (400, 1600, 512, 0, 0), (416, 1664, 768, 1, 0), (430, 1720, 768, 0, 0), (430, 1720, 3072, 1, 0), (585, 2340, 3072, 0, 0),
             (585, 2340, 3072, 1, 0), (640, 2560, 3072, 0, 0), (860, 3440, 768, 0, 0), (1050, 4200, 512, 0, 0), (1000, 4000, 768, 1, 0),
             (192, 768, 768, 0, 0), (192, 768, 3072, 0, 0), (512, 2048, 768, 0, 0)]
    got = _chosen(tmp_path, [f"mid_tiles_for_product({b}, {m}, {k}, {w}, true)" for b, m, k, w, _ in cases])
    assert [c for c, g in zip(cases, got) if g != c[4]] == []
    # operands of 2 GiB and more, which the direct-to-LDS kernels do not take
    assert _chosen(tmp_path, ["mid_tiles_for_product(288, 1152, 131136, 0, true)", "mid_tiles_for_product(288, 1152, 131136, 0, false)"]) == [1, 0]


def test_updates_over_long_sums_with_a_thin_last_pass(tmp_path):
    # (256x256 tiles, 128x128 tiles, K, 128x128 tiles are ahead)
    cases = [(144, 576, 2048, 1), (144, 576, 8192, 1), (192, 768, 2048, 1), (192, 768, 8192, 1), (187, 748, 6144, 1), (288, 1152, 2048, 1),
             (288, 1152, 16384, 1), (320, 1280, 12288, 1), (384, 1536, 16384, 1), (576, 2304, 16384, 1), (390, 1560, 2048, 1),
             (390, 1560, 8192, 1), (585, 2340, 8192, 1),
             # behind
             (144, 576, 16384, 0), (195, 780, 2048, 0), (195, 780, 4096, 0), (195, 780, 8192, 0), (196, 784, 3072, 0), (198, 792, 2048, 0),
             (216, 864, 4096, 0), (390, 1560, 12288, 0), (390, 1560, 16384, 0), (585, 2340, 16384, 0), (800, 3200, 12288, 0),
             (256, 1024, 2048, 0), (512, 2048, 4096, 0)]
    got = _chosen(tmp_path, [f"mid_tiles_for_long_update({b}, {m}, {k})" for b, m, k, _ in cases])
    assert [c for c, g in zip(cases, got) if g != c[3]] == []
