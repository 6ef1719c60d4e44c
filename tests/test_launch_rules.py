"""The rules that choose between two forms of a launch (csrc/launch_rules.h) at counts where both were measured: what was slower is not chosen.
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
    src.write_text('#include <cstdio>\n#include "launch_rules.h"\nusing namespace hydra;\nint main() {\n'
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


def test_pairs_of_an_input_gradient_and_an_update(tmp_path):
    # (input gradient's 64x64 tiles, update's, the former takes such tiles alone, too, its k, the update's, together is ahead)
    cases = [(256, 256, 1, 1024, 1024, 1), (120, 480, 1, 928, 45, 1), (1024, 192, 0, 256, 1024, 1), (640, 64, 0, 128, 1024, 1),
             (512, 256, 0, 1024, 2048, 1), (384, 64, 0, 768, 300, 1), (640, 240, 0, 512, 1024, 1), (512, 128, 0, 768, 4096, 1),
             # apart
             (576, 512, 0, 1024, 1100, 0), (576, 128, 0, 768, 1100, 0), (675, 450, 0, 952, 572, 0), (1080, 200, 0, 888, 1675, 0),
             (825, 231, 0, 664, 1567, 0), (910, 140, 0, 624, 814, 0), (930, 90, 0, 936, 1961, 0), (384, 384, 0, 976, 140, 0),
             (640, 448, 0, 432, 627, 0), (870, 210, 0, 416, 1803, 0), (440, 200, 0, 912, 692, 0), (2048, 192, 0, 256, 1024, 0),
             (256, 1280, 1, 1536, 2048, 0)]
    got = _chosen(tmp_path, [f"pair_ahead({d}, {w}, {s}, {kd}, {kw})" for d, w, s, kd, kw, _ in cases])
    assert [c for c, g in zip(cases, got) if g != c[5]] == []


def test_layernorm_backward_takes_four_workgroups_to_a_cu_for_one_pass_of_them(tmp_path):
    cases = [(768, 0), (769, 1), (826, 1), (959, 1), (1024, 1), (1025, 0), (1115, 0), (1444, 0), (1965, 0), (2340, 0)]
    assert _chosen(tmp_path, [f"ln_four_to_a_cu({b})" for b, _ in cases]) == [f for _, f in cases]


def test_layernorm_backward_of_wide_fp32_rows_asks_for_the_next_row_unless_a_few_units_hold_a_third_workgroup(tmp_path):
    cases = [(250, 2048, 1), (512, 2048, 1), (513, 2048, 0), (564, 2048, 0), (564, 2040, 0), (626, 2048, 0), (750, 2048, 1), (1024, 2048, 1),
             (564, 1536, 1), (564, 1288, 1)]
    assert _chosen(tmp_path, [f"ln_wide_ahead({b}, {d})" for b, d, _ in cases]) == [f for _, _, f in cases]


def test_layernorm_backward_of_wide_fp32_rows_where_a_few_units_hold_a_third_workgroup(tmp_path):
    cases = [(512, 1544, 1), (513, 1544, 0), (516, 1664, 0), (640, 2048, 0), (641, 2048, 1), (704, 2048, 1), (516, 1480, 1), (516, 1032, 1)]
    assert _chosen(tmp_path, [f"ln_wide_ahead({b}, {d})" for b, d, _ in cases]) == [f for _, _, f in cases]


def test_causal_attention_takes_pairs_of_row_blocks(tmp_path):
    # (row blocks of a head, of the launch, workgroups to a CU, pairs are ahead)
    cases = [(8, 768, 4, 1), (8, 768, 3, 1), (8, 2048, 3, 1), (8, 320, 2, 1), (16, 288, 4, 1), (16, 512, 2, 1), (32, 768, 2, 1), (4, 1280, 4, 1),
             (4, 640, 2, 1), (6, 3072, 3, 1), (6, 1536, 2, 1), (12, 9216, 3, 1),
             # one to a workgroup
             (16, 256, 2, 0), (4, 640, 3, 0), (4, 320, 2, 0), (6, 768, 4, 0), (6, 768, 3, 0), (6, 384, 2, 0), (2, 2048, 2, 0), (3, 3072, 3, 0),
             (5, 5120, 3, 0), (7, 7168, 2, 0), (1, 4096, 4, 0)]
    got = _chosen(tmp_path, [f"attn_pairs({n}, {b}, {c})" for n, b, c, _ in cases])
    assert [c for c, g in zip(cases, got) if g != c[3]] == []


@pytest.mark.parametrize("K,B,S,d,ffn,L,pairs", [(4, 8, 128, 256, 1024, 4, 16),   # every update but the first block's last one shares a launch
                                                 (8, 10, 110, 256, 1024, 3, 3),   # the updates of W1 only, with the gradient through Wo
                                                 (5, 4, 143, 960, 960, 3, 0), (8, 10, 110, 128, 512, 3, 12)])
def test_launches_of_a_step_that_are_shared(K, B, S, d, ffn, L, pairs):
    """Launches of a dry run against those with gradients kept, where every product is a launch of its own."""
    from hydra_workloads import configs as C, make_data
    from paper_2107_06469_amd import hydra as H
    a = [C.transformer_arch(C.KIND_ENCODER, L, d, d // 64, ffn, 64, S, 0, C.DTYPE_BF16) for _ in range(K)]
    w = C.Workload("pairs", 2, a, [C.hparams(C.OPT_ADAM, 1e-3)] * K, [[]] * K, B, S, 5, 1, 1, 3)
    data, n = make_data(w), []
    for keep in (True, False):
        ctx = H.hydra_create(dry_run=True, n_streams=1, max_group=K, keep_grads=keep)
        H.hydra_define_models(ctx, w.archs, w.hparams, 1)
        H.hydra_shard(ctx, -1, [])
        H.hydra_set_data(ctx, data["inputs"], data["target_pos"], data["targets"])
        n.append(H.hydra_train_epoch(ctx, H.SCHED_SHARD_PARALLEL, None)["launches"])
        H.hydra_destroy(ctx)
    assert n[0] - n[1] == pairs


def test_fp32_updates_over_a_small_batch_take_small_tiles_where_those_are_ahead(tmp_path):
    # (problems, M, N, K, Adam, 32x32 tiles are ahead)
    cases = [(4, 784, 768, 64, 0, 1), (4, 784, 768, 64, 1, 1), (1, 1280, 1280, 8, 0, 1), (16, 512, 512, 33, 0, 1), (16, 512, 512, 8, 1, 1), (1, 4128, 1024, 64, 1, 0),
             # SGD over up to 32 rows, 1640 tiles and more: 32x128 tiles are ahead that have most of their columns in the matrix
             (1, 1281, 1280, 32, 0, 0), (1, 1281, 1280, 33, 0, 1), (1, 1281, 1280, 32, 1, 1), (8, 512, 512, 16, 0, 0), (12, 2073, 160, 20, 0, 1), (15, 116, 1384, 10, 0, 0),
             # rows that are no whole number of lines, of 18 tile rows, 25 (a grid of 32) and 8
             (9, 554, 760, 16, 0, 0), (3, 800, 1000, 16, 0, 1), (4, 225, 2056, 32, 0, 1)]
    up = lambda n, by: (n + by - 1) // by  # noqa: E731
    calls = [f"f32_update_few({up(m, 32) * up(n, 32) * g}, {up(m, 32)}, {up(m, 32) * up(n, 128) * g}, {n}, {k}, {'true' if adam else 'false'})"
             for g, m, n, k, adam, _ in cases]
    assert [c for c, g in zip(cases, _chosen(tmp_path, calls)) if g != c[5]] == []
    # rows of whole lines, and few tile rows, keep the grid as high as the matrix, and those of which too much would be empty
    grids = ((25, 768, 1, 25), (25, 1000, 1, 32), (25, 1000, 0, 32), (24, 1000, 1, 24), (4, 1000, 1, 4), (8, 1000, 1, 8), (10, 1000, 1, 10), (11, 1000, 1, 16), (12, 1000, 0, 12),
             (18, 1000, 0, 18), (18, 1000, 1, 24), (19, 1000, 0, 24))
    assert _chosen(tmp_path, [f"f32_update_tile_rows({r}, {n}, {a})" for r, n, a, _ in grids]) == [h for *_, h in grids]
