"""End-to-end parity of the Transformer training path (encoder, heterogeneous-depth encoders, gated
causal decoder) with the CPU oracle, through the C boundary (GPU only).  bf16 tolerances as in
test_gpu_train.py: loss and parameter norms within 2e-2, plus first-step gradients (rel-L2 / cosine)
and bitwise identity across schedules and cuts."""
import hashlib
import os

import numpy as np
import pytest

from hydra_workloads import configs as C
from hydra_workloads import make_data, scaled_workload, workload
from oracle import model as OM
from oracle import optim as OO
from oracle import train as OT

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2107_06469_amd import hydra
    return hydra


def _names(arch):
    return [t[0] for t in OM.tensor_specs(arch)]


def _check_bf16(got, ref, names, p0, max_step, rel=2e-2):
    """max_step: lr * number of updates (bound on how far Adam can move one element)."""
    gl, gp = got
    rl, rp = ref
    bad = []
    lerr = float(np.max(np.abs(gl - rl) / np.abs(rl)))
    if lerr > rel:
        bad.append(f"loss rel {lerr:.2e}")
    for nm, a, b, z in zip(names, gp, rp, p0):
        a, b = a.astype(np.float64), b.astype(np.float64)
        if nm.endswith("bqkv"):
            # The key bias is a gauge parameter: adding a constant vector to every key shifts all scores of a
            # query equally, so its exact gradient is zero (rows of dS sum to zero) and the oracle never moves
            # it.  In bf16 the column sum of dk is rounding noise, which Adam turns into steps of size ~lr.
            # Those steps do not change the model's function; they are only bounded here (|step| <= lr per
            # update), and the query and value thirds are compared as usual.
            d3 = a.size // 3
            assert np.abs(b[d3:2 * d3]).max() < 1e-6, "oracle moved the key bias"
            if np.abs(a[d3:2 * d3]).max() > max_step * 1.01:
                bad.append(f"{nm}: key-bias step {np.abs(a[d3:2 * d3]).max():.3e} > {max_step:.3e}")
            keep = np.r_[0:d3, 2 * d3:3 * d3]
            a, b, z = a[keep], b[keep], z[keep]
        nb = np.linalg.norm(b)
        if abs(np.linalg.norm(a) - nb) > rel * max(nb, 1e-3):
            bad.append(f"{nm}: norm {np.linalg.norm(a):.4e} vs {nb:.4e}")
        mv, mr = np.linalg.norm(a - z), np.linalg.norm(b - z)
        if abs(mv - mr) > 5e-2 * mr + 1e-7:
            bad.append(f"{nm}: movement {mv:.3e} vs {mr:.3e}")
    assert not bad, "; ".join(bad)


@pytest.mark.parametrize("i", [2, 3, 4])
def test_scaled_transformer_workloads_match_oracle_and_schedules_agree_bitwise(H, i):
    # i=2: encoders; i=3: encoders of depth 2/4/6 with warm-up (unequal shard queues); i=4: gated causal decoders.
    # S = 48 is not a multiple of the 64-key tiles, batch*S = 144 rows and 301 classes leave ragged GEMM tiles.
    w = scaled_workload(i)
    data = make_data(w)
    ref = OT.train_all(w.archs, w.hparams, data, w.steps, w.init_seed)
    got, stats = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL)
    assert stats[0]["steps"] == w.steps
    for k in range(w.K):
        p0 = [p.astype(np.float64) for p in OM.init_params(w.archs[k], w.init_seed, k)]
        _check_bf16(got[k], ref[k], _names(w.archs[k]), p0, max_step=w.hparams[k]["lr"] * w.steps)
    variants = [dict(policy=H.SCHED_SEQUENTIAL), dict(policy=H.SCHED_SHARD_PARALLEL, cuts=[[]] * w.K, n_streams=1),
                dict(policy=H.SCHED_SHARD_PARALLEL, keep_grads=True),   # updates by update tasks, not inside gradient kernels
                dict(policy=H.SCHED_SHARD_PARALLEL, cuts=[[1]] * w.K, n_streams=2)]
    for v in variants:
        other, _ = H.train_workload(w, data, **v)
        for k in range(w.K):
            assert np.array_equal(other[k][0], got[k][0]), f"loss differs under {v}"
            for nm, a, b in zip(_names(w.archs[k]), other[k][1], got[k][1]):
                assert np.array_equal(a, b), f"{nm} differs under {v}"


@pytest.mark.parametrize("i", [2, 4])
def test_first_step_gradients_transformer(H, i):
    w = scaled_workload(i, steps=1)
    data = make_data(w)
    ctx = H.hydra_create(n_streams=2, keep_grads=True)
    H.hydra_define_models(ctx, w.archs, w.hparams, w.init_seed)
    for k in range(w.K):
        H.hydra_shard(ctx, k, w.boundaries[k])
    H.hydra_set_data(ctx, data["inputs"], data["target_pos"], data["targets"])
    H.hydra_train_epoch(ctx)
    bad = []
    for k in range(w.K):
        g = H.hydra_read_grads(ctx, k)
        p0 = OM.init_params(w.archs[k], w.init_seed, k)
        _, gref = OM.loss_and_grads(w.archs[k], p0, OT.batch_at(data, 1))
        for nm, a, b in zip(_names(w.archs[k]), g, gref):
            a, b = a.astype(np.float64).reshape(-1), b.reshape(-1)
            rel = np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)
            cos = float(a @ b) / max(np.linalg.norm(a) * np.linalg.norm(b), 1e-30)
            if rel > 3e-2 or cos < 0.999:
                bad.append(f"model {k} {nm}: rel {rel:.3e} cos {cos:.5f}")
    H.hydra_destroy(ctx)
    assert not bad, "; ".join(bad)


@pytest.mark.parametrize("batch,seq,d,heads,ffn,vocab", [(2, 40, 64, 1, 136, 70), (8, 128, 128, 2, 512, 301), (9, 120, 128, 2, 264, 96), (3, 130, 256, 4, 1024, 64)])
def test_paired_gradient_launches_keep_the_bits_of_separate_ones(H, batch, seq, d, heads, ffn, vocab):
    """Small weight gradients with their update share a launch with the next input gradient (both tile shapes of the update: sums of up to
    1024 tokens and longer ones); with gradients kept every product is a launch of its own.  Losses and parameters are the same bits, and
    the paired run has fewer launches."""
    archs = [C.transformer_arch(C.KIND_ENCODER, 2, d, heads, ffn, vocab, seq, 0, C.DTYPE_BF16) for _ in range(2)]
    w = C.Workload("encoder_pairs", 2, archs, [C.hparams(C.OPT_ADAM, 1e-3), C.hparams(C.OPT_SGD, 1e-2)], [[1]] * 2, batch, seq, 5, 3, 3, 31 + seq)
    data = make_data(w)
    paired, ps = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL)
    apart, as_ = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL, keep_grads=True)
    assert ps[0]["launches"] < as_[0]["launches"]
    for k in range(w.K):
        assert np.array_equal(paired[k][0], apart[k][0])
        for a, b in zip(paired[k][1], apart[k][1]):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("gated,recompute", [(1, False), (1, True), (0, True)])
@pytest.mark.parametrize("batch,seq,d,heads,ffn", [(3, 48, 128, 2, 344), (9, 120, 128, 1, 264)])
def test_paired_gradient_launches_of_gated_decoders_and_recomputed_blocks(H, gated, recompute, batch, seq, d, heads, ffn):
    """As above where a held W1 gradient rides with the gradient through Wg, which reads and writes its own output, and where the products'
    operands lie in workspaces that the shards' tasks share."""
    kind = C.KIND_DECODER if gated else C.KIND_ENCODER
    archs = [C.transformer_arch(kind, 4, d, heads, ffn, 96, seq, gated, C.DTYPE_BF16) for _ in range(2)]
    n_targets = seq if gated else 5
    w = C.Workload("paired", 2, archs, [C.hparams(C.OPT_ADAM, 1e-3), C.hparams(C.OPT_SGD, 1e-2)], [[2]] * 2, batch, seq, n_targets, 3, 3, 31 + seq)
    data = make_data(w)
    # room for one shard's workspace, or a few
    kw = dict(activation_budget_bytes=max(3 << 20, batch * seq * 13000)) if recompute else {}
    paired, ps = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL, **kw)
    apart, as_ = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL, keep_grads=True)
    if recompute:                                                        # the forward passes of the shards but the last run twice
        kept, ks = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL, keep_grads=True, **kw)
        assert ks[0]["launches"] > as_[0]["launches"] and ps[0]["launches"] < ks[0]["launches"]
    else:
        assert ps[0]["launches"] < as_[0]["launches"]
    for k in range(w.K):
        assert np.array_equal(paired[k][0], apart[k][0])
        for a, b in zip(paired[k][1], apart[k][1]):
            assert np.array_equal(a, b)


def test_data_is_validated(H):
    w = scaled_workload(2, K=1)
    d = make_data(w)
    ctx = H.hydra_create(n_streams=1)
    H.hydra_define_models(ctx, w.archs, w.hparams, w.init_seed)
    H.hydra_shard(ctx, -1, [])
    ids = d["inputs"].copy()
    ids[0, 0, 0] = 301
    with pytest.raises(H.HydraError):
        H.hydra_set_data(ctx, ids, d["target_pos"], d["targets"])
    pos = d["target_pos"].copy()
    pos[0, 0, 1] = pos[0, 0, 0]
    with pytest.raises(H.HydraError):
        H.hydra_set_data(ctx, d["inputs"], pos, d["targets"])
    H.hydra_set_data(ctx, d["inputs"], d["target_pos"], d["targets"])
    H.hydra_destroy(ctx)


def test_config2_full_size_one_step_sampled_against_oracle(H):
    """Full-size workload 2 (K=4 encoders, 12 blocks, d=768, 12 heads, S=512, batch 32, vocabulary 30522) in the
    benchmark's launch configuration for one step; the oracle recomputes the first loss of one model
    (forward only, fp64) and all four first losses must sit near ln(30522)."""
    w = workload(2)
    w.steps = w.n_batches = 1
    data = make_data(w)
    got, stats = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL)
    k = 1
    params = OM.init_params(w.archs[k], w.init_seed, k)
    x, batch = None, OT.batch_at(data, 1)
    for u in range(OM.n_units(w.archs[k])):
        x, _ = OM.unit_fwd(w.archs[k], params, u, x, batch)
    assert abs(got[k][0][0] - float(x)) <= 2e-2 * float(x)
    for kk in range(w.K):
        assert abs(got[kk][0][0] - np.log(30522)) < 0.3
        assert all(np.all(np.isfinite(p)) for p in got[kk][1])


def test_config3_full_size_one_step_sampled_against_oracle(H):
    """Full-size workload 3 (K=16 encoders of depth 12/18/24, d=1024, 16 heads, S=512, batch 16, vocabulary 32000,
    shards of 6 blocks: 2, 3 or 4 shards per model, i.e. unequal shard queues) for one step in the benchmark's launch
    configuration.  The oracle recomputes the first loss of one 12-block model (forward only, fp64); every first
    loss must be finite and sit near ln(32000); models of equal depth share launch groups."""
    w = workload(3)
    w.steps = w.n_batches = 1
    data = make_data(w)
    got, stats = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL)
    depths = w.extra["depths"]
    assert set(depths) == {12, 18, 24}
    assert stats[0]["grouped_tasks"] > 0
    k = depths.index(12)
    params = OM.init_params(w.archs[k], w.init_seed, k)
    x, batch = None, OT.batch_at(data, 1)
    for u in range(OM.n_units(w.archs[k])):
        x, _ = OM.unit_fwd(w.archs[k], params, u, x, batch)
    assert abs(got[k][0][0] - float(x)) <= 2e-2 * float(x)
    for kk in range(w.K):
        assert abs(got[kk][0][0] - np.log(32000)) < 0.4
        assert all(np.all(np.isfinite(p)) for p in got[kk][1])


def _first_step_against_oracle(H, w, k, batch):
    """Full-width models on `batch` sequences per step, all K models in the benchmark's launch configuration.
    Step 1: every gradient tensor of model k against the oracle's (relative L2 and cosine), the loss, and the
    parameters after the update (norms, and how far each tensor moved); step 2, on a new batch: the loss."""
    w.batch, w.steps, w.n_batches = batch, 2, 2
    data = make_data(w)
    one = lambda i: {n: (None if v is None else v[i:i + 1]) for n, v in data.items()}
    arch, hp, names = w.archs[k], w.hparams[k], _names(w.archs[k])
    # GPU, gradients kept: first-step gradients
    ctx = H.hydra_create(n_streams=4, keep_grads=True)
    try:
        H.hydra_define_models(ctx, w.archs, w.hparams, w.init_seed)
        for kk in range(w.K):
            H.hydra_shard(ctx, kk, w.boundaries[kk])
        H.hydra_set_data(ctx, one(0)["inputs"], one(0)["target_pos"], one(0)["targets"])
        H.hydra_train_epoch(ctx)
        grads = H.hydra_read_grads(ctx, k)
    finally:
        H.hydra_destroy(ctx)
    # GPU, the default placement (updates inside the gradient kernels): two steps, parameters read after the first
    ctx = H.hydra_create(n_streams=4)
    try:
        H.hydra_define_models(ctx, w.archs, w.hparams, w.init_seed)
        for kk in range(w.K):
            H.hydra_shard(ctx, kk, w.boundaries[kk])
        H.hydra_set_data(ctx, one(0)["inputs"], one(0)["target_pos"], one(0)["targets"])
        st = H.hydra_train_epoch(ctx)
        assert st["grouped_tasks"] > 0
        p1 = H.hydra_read_params(ctx, k)
        H.hydra_set_data(ctx, one(1)["inputs"], one(1)["target_pos"], one(1)["targets"])
        H.hydra_train_epoch(ctx)
        losses = H.hydra_read_loss(ctx, k)
        others = [H.hydra_read_loss(ctx, kk) for kk in range(w.K)]
    finally:
        H.hydra_destroy(ctx)
    assert len(losses) == 2 and all(np.all(np.isfinite(l)) for l in others)
    # oracle: one forward + backward + update, then a forward on the second batch
    p0 = OM.init_params(arch, w.init_seed, k)
    l1, gref = OM.loss_and_grads(arch, p0, OT.batch_at(data, 1))
    bad = []
    for nm, a, b in zip(names, grads, gref):
        a, b = a.astype(np.float64).reshape(-1), b.reshape(-1)
        if nm.endswith("bqkv"):      # the key third has an exactly zero gradient (softmax shift invariance); compare q and v
            d3 = a.size // 3
            assert np.abs(b[d3:2 * d3]).max() < 1e-12
            a, b = np.r_[a[:d3], a[2 * d3:]], np.r_[b[:d3], b[2 * d3:]]
        rel = np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)
        cos = float(a @ b) / max(np.linalg.norm(a) * np.linalg.norm(b), 1e-30)
        if rel > 3e-2 or cos < 0.999:
            bad.append(f"{nm}: rel {rel:.3e} cos {cos:.5f}")
    assert not bad, "; ".join(bad)
    ref = [p.copy() for p in p0]
    state = OO.new_state(ref)
    for j, g in enumerate(gref):
        OO.update_tensor(hp, 1, ref[j], g, state["m"][j], state["v"][j])
    x, b2 = None, OT.batch_at(data, 2)
    for u in range(OM.n_units(arch)):
        x, _ = OM.unit_fwd(arch, ref, u, x, b2)
    lr1 = hp["lr"] * (min(1.0, 1.0 / hp["warmup_steps"]) if hp["warmup_steps"] > 0 else 1.0)
    _check_bf16((losses.astype(np.float64), p1), (np.array([l1, float(x)]), ref), names,
                [p.astype(np.float64) for p in p0], max_step=lr1)


def test_config2_full_width_first_step_gradients_and_update_against_oracle(H):
    """Workload 2's encoders at full width (12 blocks, d=768, 12 heads, FFN 3072, S=512, vocabulary 30522, K=4, 3 shards)
    on 8 sequences per step instead of 32, which is what the fp64 oracle finishes in a test: 4096 tokens, so the
    weight gradients of the 768-wide matrices still run as split sums (4 ranges), attention has 8 key tiles per block
    and the head is 608 target rows x 30522 classes."""
    _first_step_against_oracle(H, workload(2), k=1, batch=8)


def test_config3_full_width_first_step_gradients_and_update_against_oracle(H):
    """Workload 3's encoders at full width (d=1024, 16 heads, FFN 4096, S=512, vocabulary 32000, K=16 models of depth
    12/18/24 in shards of 6 blocks, warm-up grid) on 4 sequences per step instead of 16; the sampled model is the first
    one of depth 12."""
    w = workload(3)
    _first_step_against_oracle(H, w, k=w.extra["depths"].index(12), batch=4)


def training_bits(H, i):
    """Digest of the losses and trained parameters of all models of scaled workload i."""
    w = scaled_workload(i)
    got, _ = H.train_workload(w, make_data(w), H.SCHED_SHARD_PARALLEL)
    h = hashlib.sha256()
    for losses, params in (got[k] for k in range(w.K)):
        h.update(np.ascontiguousarray(losses).tobytes())
        for p in params:
            h.update(np.ascontiguousarray(p).tobytes())
    return h.hexdigest()[:32]


@pytest.mark.parametrize("i", [2, 3, 4])
def test_training_keeps_its_bits(H, i):
    """A training run gives the same parameters, bit for bit, whatever version of the kernels runs it (digests recorded on an MI355X
    before attention and the LayerNorm backward pass were rewritten).  A change of rounding that is meant needs new digests."""
    with open(os.path.join(os.path.dirname(__file__), "golden", "training_bits.txt")) as f:
        want = dict(ln.split() for ln in f if not ln.startswith("#"))
    assert training_bits(H, i) == want[str(i)]
