"""Schedules and drivers beyond the three basic policies (GPU only): the task-parallel policy, models dropped
from the schedule by model selection, the automatic sharder, and workloads with the shapes the paper's own
evaluation names.  Everything must reproduce the bits of the plain shard-parallel run (the paper's third
desideratum) or match the oracle within the tolerances of test_gpu_train.py."""
import numpy as np
import pytest

from hydra_workloads import configs as C
from hydra_workloads import make_data, paper_shaped_workload, scaled_workload
from oracle import model as OM
from oracle import train as OT

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2107_06469_amd import hydra
    return hydra


def _oracle_parity_bf16(w, got, data, steps, models, rel=2e-2):
    """The bf16 tolerances of the end-to-end tests against the oracle's unsharded, one-model-at-a-time training:
    per-step loss and parameter norms within 2e-2, parameter movement within 5e-2 (the key third of bqkv, whose exact
    gradient is zero, is bounded by lr per step instead)."""
    ref = OT.train_all(w.archs, w.hparams, data, steps, w.init_seed, models=models)
    for k in models:
        gl, gp = got[k]
        rl, rp = ref[k]
        assert len(gl) == steps and np.all(np.abs(gl - rl) <= rel * np.abs(rl)), f"model {k} loss: {gl} vs {rl}"
        p0 = OM.init_params(w.archs[k], w.init_seed, k)
        for (nm, _, _), a, b, z in zip(OM.tensor_specs(w.archs[k]), gp, rp, p0):
            a, b, z = a.astype(np.float64), b.astype(np.float64), z.astype(np.float64)
            if nm.endswith("bqkv"):
                d3 = a.size // 3
                assert np.abs(a[d3:2 * d3]).max() <= 1.01 * w.hparams[k]["lr"] * steps, f"model {k} {nm}: key bias"
                keep = np.r_[0:d3, 2 * d3:3 * d3]
                a, b, z = a[keep], b[keep], z[keep]
            nb = np.linalg.norm(b)
            assert abs(np.linalg.norm(a) - nb) <= rel * max(nb, 1e-3), f"model {k} {nm}: norm"
            mv, mr = np.linalg.norm(a - z), np.linalg.norm(b - z)
            assert abs(mv - mr) <= 5e-2 * mr + 1e-7, f"model {k} {nm}: movement {mv} vs {mr}"


def _same(got, ref, what, models=None):
    for k in (models if models is not None else ref):
        assert np.array_equal(got[k][0], ref[k][0]), f"loss of model {k} differs ({what})"
        for a, b in zip(got[k][1], ref[k][1]):
            assert np.array_equal(a, b), f"parameters of model {k} differ ({what})"


@pytest.mark.parametrize("i", [1, 3])
def test_task_parallel_policy_reproduces_the_shard_parallel_bits(H, i):
    w = scaled_workload(i, steps=3)
    data = make_data(w)
    ref, rs = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL)
    for n_streams in (1, 3, 4):
        got, st = H.train_workload(w, data, H.SCHED_TASK_PARALLEL, n_streams=n_streams)
        assert st[0]["grouped_tasks"] == 0 and st[0]["launches"] > rs[0]["launches"]
        _same(got, ref, f"task-parallel, {n_streams} streams")
    _oracle_parity_bf16(w, got, data, w.steps, list(range(w.K)))      # and the task-parallel result is the oracle's
    if i == 3:  # with spilled state and recomputed activations as well
        nb = [sum((r * c + 63) // 64 * 64 for r, c in sh) for sh in _shapes(H, w)]
        budget = sum(nb) * 2 + 256 * 1024 + int(2.5 * (max(nb) // 2 * 16 + 64 * 1024))
        got, st = H.train_workload(w, data, H.SCHED_TASK_PARALLEL, device_budget_bytes=budget, activation_budget_bytes=4 << 20)
        assert st[0]["h2d_bytes"] > 0
        _same(got, ref, "task-parallel, spilled and recomputed")


def _shapes(H, w):
    ctx = H.hydra_create(dry_run=True)
    H.hydra_define_models(ctx, w.archs, w.hparams, w.init_seed)
    out = [H.hydra_tensor_shapes(ctx, k) for k in range(w.K)]
    H.hydra_destroy(ctx)
    return out


def _epochs(H, w, data, n_epochs, drop=None, policy=None):
    """Trains n_epochs; drop = {epoch: [models]} marks models inactive before that epoch."""
    ctx = H.hydra_create(n_streams=4)
    try:
        H.hydra_define_models(ctx, w.archs, w.hparams, w.init_seed)
        for k in range(w.K):
            H.hydra_shard(ctx, k, w.boundaries[k])
        H.hydra_set_data(ctx, data["inputs"], data["target_pos"], data["targets"])
        for e in range(n_epochs):
            for k in (drop or {}).get(e, []):
                H.hydra_set_active(ctx, k, False)
            H.hydra_train_epoch(ctx, H.SCHED_SHARD_PARALLEL if policy is None else policy)
        return {k: (H.hydra_read_loss(ctx, k), H.hydra_read_params(ctx, k)) for k in range(w.K)}
    finally:
        H.hydra_destroy(ctx)


def test_dropping_models_leaves_the_others_unchanged(H):
    w = scaled_workload(2, K=4, depths=[4, 4, 4, 4], steps=2)
    data = make_data(w)
    full = _epochs(H, w, data, 3)
    part = _epochs(H, w, data, 3, drop={1: [1], 2: [3]})
    _same(part, full, "models 0 and 2 while 1 and 3 drop out", models=[0, 2])
    one = _epochs(H, w, data, 1)
    two = _epochs(H, w, data, 2)
    _same(part, one, "model 1 stopped after one epoch", models=[1])
    _same(part, two, "model 3 stopped after two epochs", models=[3])
    # against the oracle: every model trained alone, unsharded, for as many steps as it stayed in the schedule
    # (the batches cycle: epoch e uses the same w.steps batches again)
    for k, n_ep in ((0, 3), (1, 1), (2, 3), (3, 2)):
        _oracle_parity_bf16(w, part, data, n_ep * w.steps, [k])


def test_successive_halving_keeps_the_best_configuration(H):
    from paper_2107_06469_amd import selection
    w = scaled_workload(1, K=4, steps=4, dtype=C.DTYPE_F32)
    lrs = [3e-3, 1e-6, 1e-3, 1e-7]                       # two configurations that learn, two that barely move
    for h, lr in zip(w.hparams, lrs):
        h["lr"] = lr
    w.n_batches = 1                                      # one batch repeated: the loss falls as it is memorised
    data = make_data(w)
    ctx = H.hydra_create(n_streams=4)
    try:
        H.hydra_define_models(ctx, w.archs, w.hparams, w.init_seed)
        H.hydra_shard(ctx, -1, w.boundaries[0])
        H.hydra_set_data(ctx, data["inputs"], None, data["targets"])
        res = selection.successive_halving(ctx, w.K, epochs_per_rung=3)
        assert len(res["survivors"]) == 1 and res["survivors"][0] in (0, 2)
        assert sorted(s["model"] for s in res["stopped"] if s["rung"] == 0) == [1, 3]
        assert [len(r["models"]) for r in res["rungs"]] == [4, 2, 1]
        best = res["survivors"][0]
        losses = H.hydra_read_loss(ctx, best)
        assert len(losses) == 9 and losses[-1] < losses[0]
        assert len(H.hydra_read_loss(ctx, 1)) == 3
    finally:
        H.hydra_destroy(ctx)
    # the survivor's run is the run it would have had alone
    plain = _epochs(H, w, data, 9)
    assert np.array_equal(plain[best][0], losses)


def test_automatic_cuts_train_to_the_same_bits(H):
    w = scaled_workload(2, K=2, depths=[6, 6], steps=2)
    data = make_data(w)
    ref, _ = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL)
    ctx = H.hydra_create(n_streams=4)
    try:
        H.hydra_define_models(ctx, w.archs, w.hparams, w.init_seed)
        cuts = H.hydra_auto_shard(ctx, 0, n_shards=3)
        H.hydra_auto_shard(ctx, 1, n_shards=2)
        assert len(cuts) == 2 and H.hydra_shard_count(ctx, 1) == 2
        H.hydra_set_data(ctx, data["inputs"], data["target_pos"], data["targets"])
        H.hydra_train_epoch(ctx, H.SCHED_SHARD_PARALLEL)
        got = {k: (H.hydra_read_loss(ctx, k), H.hydra_read_params(ctx, k)) for k in range(w.K)}
    finally:
        H.hydra_destroy(ctx)
    _same(got, ref, "automatic cuts")
    _oracle_parity_bf16(w, got, data, w.steps, [0, 1])                # the oracle knows no cuts at all


def test_paper_shaped_feed_forward_net_sharded_equals_unsharded_and_matches_oracle(H):
    """The paper's equivalence experiment (Evaluation, "Workloads": a 1.2 M-parameter feed-forward net trained sharded
    and on a single device must give the same result), on synthetic rows: 3 epochs over 4 batches, fp32, SGD."""
    w = paper_shaped_workload("ffn_1p2m")
    assert C.param_count(w.archs[0]) == 1201162
    data = make_data(w)
    sharded, st = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL, epochs=3)
    assert [s["steps"] for s in st] == [4, 4, 4]
    whole, _ = H.train_workload(w, data, H.SCHED_SEQUENTIAL, epochs=3, cuts=[[]] * w.K)
    _same(whole, sharded, "unsharded, one model after another")
    ref = OT.train_all(w.archs, w.hparams, data, w.steps, w.init_seed)
    for k in range(w.K):
        gl, gp = sharded[k]
        rl, rp = ref[k]
        assert np.all(np.abs(gl - rl) <= 1e-5 * np.abs(rl)), (k, gl, rl)
        for a, b in zip(gp, rp):
            b = b.astype(np.float64)
            scale = max(float(np.abs(b).max()), 1e-2)
            err = float(np.linalg.norm(a - b)) / max(float(np.linalg.norm(b)), 1e-2)
            assert err <= 1e-5 and np.abs(a - b).max() <= 1e-5 * scale, (k, a.shape, err, np.abs(a - b).max())


def test_bert_large_shaped_encoders_one_step_against_oracle(H):
    """BERT-Large-shaped encoders (24 blocks, d=1024, 16 heads, FFN 4096, 384-token sequences: the shape of the
    paper's large workload, Evaluation, "Workloads") on synthetic tokens, two configurations, four shards each, one
    step; the oracle recomputes the first loss of model 1 (forward only, fp64)."""
    w = paper_shaped_workload("bert_large_384", K=2)
    w.batch, w.steps, w.n_batches = 4, 1, 1
    data = make_data(w)
    got, st = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL)
    assert st[0]["grouped_tasks"] == 2 * 4 * 3
    k = 1
    params = OM.init_params(w.archs[k], w.init_seed, k)
    x, batch = None, OT.batch_at(data, 1)
    for u in range(OM.n_units(w.archs[k])):
        x, _ = OM.unit_fwd(w.archs[k], params, u, x, batch)
    assert abs(got[k][0][0] - float(x)) <= 2e-2 * float(x)
    for kk in range(w.K):
        assert abs(got[kk][0][0] - np.log(30522)) < 0.4
        assert all(np.all(np.isfinite(p)) for p in got[kk][1])


def test_profile_accounts_the_algorithmic_work_of_an_epoch(H):
    """The per-kernel-class counters behind the benchmark's rates: an epoch of workload 0 (4 ReLU MLPs, 256 wide,
    4 hidden layers + a 10-way head, batch 32, 10 steps, SGD) must be booked with the products' 2·m·n·k each."""
    w = C.workload(0)
    data = make_data(w)
    ctx = H.hydra_create(n_streams=4)
    try:
        H.hydra_define_models(ctx, w.archs, w.hparams, w.init_seed)
        for k in range(w.K):
            H.hydra_shard(ctx, k, w.boundaries[k])
        H.hydra_set_data(ctx, data["inputs"], data["target_pos"], data["targets"])
        assert len(H.hydra_tensor_shapes(ctx, 0)) == 2 * 5             # weight and bias of 5 layers
        H.hydra_train_epoch(ctx, H.SCHED_SHARD_PARALLEL, None)          # profiling off: nothing booked
        assert H.hydra_profile_read(ctx) == {}
        H.hydra_profile_enable(ctx, True)
        steps = H.hydra_train_epoch(ctx, H.SCHED_SHARD_PARALLEL, None)["steps"]
        assert steps == w.n_batches
        prof = H.hydra_profile_read(ctx, reset=False)
        layers = [(256, 256)] * 4 + [(256, 10)]
        per_step = lambda ls: sum(2.0 * w.batch * i * o for i, o in ls) * w.K
        assert prof["gemm_fwd"]["flops"] == pytest.approx(per_step(layers) * steps, rel=1e-12)
        assert prof["gemm_dgrad"]["flops"] == pytest.approx(per_step(layers[1:]) * steps, rel=1e-12)  # no dX of the input
        wg = sum(prof[c]["flops"] for c in ("gemm_wgrad", "wgrad_update") if c in prof)
        assert wg == pytest.approx(per_step(layers) * steps, rel=1e-12)
        # fused SGD update in fp32: the weight read and written (8 B) plus the two operands of the product
        upd = sum((8.0 * i * o + 4.0 * w.batch * (i + o)) for i, o in layers) * w.K * steps
        assert prof["wgrad_update"]["bytes"] == pytest.approx(upd, rel=1e-12)
        for c, p in prof.items():
            assert p["launches"] > 0 and p["total_ms"] > 0.0, c
        assert H.hydra_profile_read(ctx, reset=True) == prof             # reading with reset returns, then clears
        assert H.hydra_profile_read(ctx) == {}
        H.hydra_profile_enable(ctx, False)
        H.hydra_train_epoch(ctx, H.SCHED_SHARD_PARALLEL, None)
        assert H.hydra_profile_read(ctx) == {}
    finally:
        H.hydra_destroy(ctx)


@pytest.mark.parametrize("i", [2, 4])
def test_profile_accounts_the_products_of_transformer_blocks(H, i):
    """Encoders (workload 2's layers) and gated causal decoders (workload 4's) at reduced size: every weight matrix
    is booked once per pass with 2·rows·in·out, the attention products with 4 (forward) + 10 (backward) ·B·S²·d,
    halved under the causal mask; every weight's update with the state's bytes and its product's operands, also where it shares a
    launch with an input gradient."""
    w = scaled_workload(i, K=2, depths=[2, 4], steps=2)
    data = make_data(w)
    ctx = H.hydra_create(n_streams=2)
    try:
        H.hydra_define_models(ctx, w.archs, w.hparams, w.init_seed)
        for k in range(w.K):
            H.hydra_shard(ctx, k, w.boundaries[k])
        H.hydra_set_data(ctx, data["inputs"], data["target_pos"], data["targets"])
        H.hydra_profile_enable(ctx, True)
        steps = H.hydra_train_epoch(ctx, H.SCHED_SHARD_PARALLEL, None)["steps"]
        prof = H.hydra_profile_read(ctx)
        T, NT = w.batch * w.seq, w.batch * w.n_targets
        gemm = att = upd = 0.0
        for a in w.archs:
            d, F, V, L = a["d_model"], a["d_ffn"], a["n_out"], a["n_layers"]
            # fused Adam update: p, m, v read and written, the bf16 copy written (26 B); the product's two bf16 operands
            mats = [(3 * d, d), (d, d), (F, d), (d, F)] + [(F, d)] * a["ffn_gated"]
            upd += sum(26.0 * o * i + 2.0 * T * (o + i) for o, i in mats) * L + 26.0 * V * d + 2.0 * NT * (V + d)
            gemm += 2.0 * T * L * (3 * d * d + d * d + (3 if a["ffn_gated"] else 2) * d * F) + 2.0 * NT * d * V
            att += w.batch * float(w.seq) ** 2 * d * L * (0.5 if a["causal"] else 1.0)
        assert prof["gemm_fwd"]["flops"] == pytest.approx(gemm * steps, rel=1e-12)
        assert prof["gemm_dgrad"]["flops"] == pytest.approx(gemm * steps, rel=1e-12)
        wg = sum(prof[c]["flops"] for c in ("gemm_wgrad", "wgrad_update") if c in prof)
        assert wg == pytest.approx(gemm * steps, rel=1e-12)
        assert prof["wgrad_update"]["bytes"] == pytest.approx(upd * steps, rel=1e-12)
        assert prof["attention"]["flops"] == pytest.approx(14.0 * att * steps, rel=1e-12)
    finally:
        H.hydra_destroy(ctx)


def test_automatic_budgets_reproduce_the_resident_bits_and_the_oracle(H):
    """auto_budget plans spilling and recomputation from the device capacity it is given: with room for the state but
    not the activations it recomputes, with less than the state it spills as well; either way every bit equals the
    run that keeps everything resident, which in turn matches the oracle."""
    w = scaled_workload(4, K=3, depths=[4, 4, 4], steps=3, batch=8, seq=128)
    data = make_data(w)
    ref, rs = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL)
    nb = [sum((r * c + 63) // 64 * 64 for r, c in sh) for sh in _shapes(H, w)]
    state = sum(nb) * 18
    acts = rs[0]["peak_dev_bytes"] - state
    assert acts > state
    got, st = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL, auto_budget=True, device_capacity_bytes=state + acts // 2)
    assert st[0]["h2d_bytes"] == 0 and st[0]["launches"] > rs[0]["launches"] and st[0]["peak_dev_bytes"] < rs[0]["peak_dev_bytes"]
    _same(got, ref, "automatic budgets: recomputed activations")
    got, st = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL, auto_budget=True, device_capacity_bytes=int(state * 0.9))
    assert st[0]["h2d_bytes"] > 0 and st[0]["peak_dev_bytes"] <= int(state * 0.9)
    _same(got, ref, "automatic budgets: spilled state and recomputed activations")
    got, st = H.train_workload(w, data, H.SCHED_SHARD_PARALLEL, auto_budget=True)      # the real device: room for everything
    assert st[0]["h2d_bytes"] == 0 and st[0]["launches"] == rs[0]["launches"]
    _same(got, ref, "automatic budgets on the whole device")
    _oracle_parity_bf16(w, ref, data, w.steps, [0, 1, 2])


@pytest.mark.parametrize("case", ["mlp_bf16_adam", "mlp_f32_sgd_small", "encoder_warmup", "decoder_spilled"])
def test_training_resumed_from_a_checkpoint_continues_bit_for_bit(H, case):
    """Two epochs in one context against one epoch, then parameters, moments and step counts exported, imported into
    a fresh context and a second epoch there: same losses and parameters, bit for bit (Adam's bias corrections and the
    warm-up depend on the step count; spilled state lives in host memory)."""
    budget = 0
    if case == "mlp_bf16_adam":
        w = scaled_workload(1, K=3, steps=3)
    elif case == "mlp_f32_sgd_small":
        w = C.workload(0)
        w.steps = w.n_batches = 4
    elif case == "encoder_warmup":
        w = scaled_workload(3, K=3, steps=3, warmup=4)
    else:
        w = scaled_workload(4, K=2, depths=[4, 4], steps=3)
        nb = [sum((r * c + 63) // 64 * 64 for r, c in sh) for sh in _shapes(H, w)]
        budget = sum(nb) * 2 + 256 * 1024 + int(2.5 * (max(nb) // 2 * 16 + 64 * 1024))
    data = make_data(w)

    def fresh():
        ctx = H.hydra_create(n_streams=4, device_budget_bytes=budget)
        H.hydra_define_models(ctx, w.archs, w.hparams, w.init_seed)
        for k in range(w.K):
            H.hydra_shard(ctx, k, w.boundaries[k])
        H.hydra_set_data(ctx, data["inputs"], data["target_pos"], data["targets"])
        return ctx
    a = fresh()
    try:
        H.hydra_train_epoch(a)
        saved = [(H.hydra_read_params(a, k), H.hydra_read_optimizer_state(a, k)) for k in range(w.K)]
        H.hydra_train_epoch(a)
        want = {k: (H.hydra_read_loss(a, k), H.hydra_read_params(a, k)) for k in range(w.K)}
    finally:
        H.hydra_destroy(a)
    b = fresh()
    try:
        for k, (params, (m, v, steps)) in enumerate(saved):
            assert steps == w.steps and (m.size == 0) == (w.hparams[k]["opt"] == C.OPT_SGD)
            H.hydra_write_params(b, k, -1, params)
            H.hydra_write_optimizer_state(b, k, m, v, steps)
        H.hydra_train_epoch(b)
        for k in range(w.K):
            assert np.array_equal(H.hydra_read_loss(b, k), want[k][0][w.steps:]), f"{case}: loss of model {k}"
            for x, y in zip(H.hydra_read_params(b, k), want[k][1]):
                assert np.array_equal(x, y), f"{case}: parameters of model {k}"
    finally:
        H.hydra_destroy(b)
