"""Parity of the Transformer-side HIP operations (LayerNorm, attention, embedding) with the oracle's
layer functions (GPU only).  bf16 inputs are rounded once on the host and the oracle gets exactly those
values in fp64; tolerances are the bf16 output rounding (2^-8 relative) plus, for attention, the bf16
rounding of the probabilities that feed the second matrix product."""
import hashlib
import math
import os

import numpy as np
import pytest

from oracle import layers as OL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a HIP device"
    return t


@pytest.fixture(scope="module")
def ops():
    from paper_2107_06469_amd import ops as o
    return o


def _bf(torch, a):
    """fp array -> (bf16 cuda tensor, the rounded values as fp64)."""
    t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(torch.bfloat16)
    return t.cuda(), t.to(torch.float64).numpy()


def _f32(torch, a):
    t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32))
    return t.cuda(), t.to(torch.float64).numpy()


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("shape", [(37, 64), (130, 768), (9, 1024), (5, 2048 + 64), (6, 4096), (100, 1536), (70, 4096)])
def test_layernorm_forward_and_backward(torch, ops, dtype, shape):
    rows, d = shape
    r = np.random.default_rng(rows * d)
    mk = _bf if dtype else _f32
    tdt = torch.bfloat16 if dtype else torch.float32
    G = 2
    xs, ys, gs, bs, mus, rss, dys, adds, dxs, parts, dgs, dbs, ref = ([] for _ in range(13))
    for g in range(G):
        xd, xv = mk(torch, r.normal(size=(rows, d)) * 2 + 0.5)
        dyd, dyv = mk(torch, r.normal(size=(rows, d)))
        ad, av = mk(torch, r.normal(size=(rows, d)))
        gam, bet = (r.normal(size=d) * 0.3 + 1).astype(np.float32), (r.normal(size=d) * 0.2).astype(np.float32)
        xs.append(xd), dys.append(dyd), adds.append(ad)
        gs.append(torch.from_numpy(gam).cuda()), bs.append(torch.from_numpy(bet).cuda())
        ys.append(torch.zeros((rows, d), dtype=tdt, device="cuda"))
        dxs.append(torch.zeros((rows, d), dtype=tdt, device="cuda"))
        mus.append(torch.zeros(rows, device="cuda")), rss.append(torch.zeros(rows, device="cuda"))
        parts.append(torch.zeros(ops.hydra_op_layernorm_part_floats(rows, d), device="cuda"))
        dgs.append(torch.zeros(d, device="cuda")), dbs.append(torch.zeros(d, device="cuda"))
        y, cache = OL.layernorm_fwd(xv, gam.astype(np.float64), bet.astype(np.float64))
        dx, dg, db = OL.layernorm_bwd(dyv, cache, gam.astype(np.float64))
        ref.append((y, cache, dx + av, dg, db))
    ops.hydra_op_layernorm_fwd(dtype, rows, d, d, 1e-5, xs, ys, gs, bs, mus, rss)
    ops.hydra_op_layernorm_bwd(dtype, rows, d, d, xs, dys, adds, dxs, gs, mus, rss, parts, dgs, dbs)
    torch.cuda.synchronize()
    out_eps = 2.0 ** -8 if dtype else 2e-6
    for g in range(G):
        y, (xhat, rstd), dx, dg, db = ref[g]
        assert np.allclose(mus[g].cpu().numpy(), (xs[g].double().cpu().numpy()).mean(-1), atol=1e-5)
        assert np.allclose(rss[g].cpu().numpy(), rstd[:, 0], rtol=2e-5)
        assert np.all(np.abs(ys[g].double().cpu().numpy() - y) <= out_eps * np.abs(y) + 1e-5)
        assert np.all(np.abs(dxs[g].double().cpu().numpy() - dx) <= out_eps * np.abs(dx) + 2e-5)
        # column sums over `rows` terms in fp32
        assert np.allclose(dgs[g].cpu().numpy(), dg, rtol=1e-4, atol=1e-4 * math.sqrt(rows))
        assert np.allclose(dbs[g].cpu().numpy(), db, rtol=1e-4, atol=1e-4 * math.sqrt(rows))


def _attention_case(torch, ops, B, S, H, DH, causal, seed):
    r = np.random.default_rng(seed)
    d = H * DH
    G = 2
    qkvs, os_, lses, douts, deltas, dqkvs, refs = [], [], [], [], [], [], []
    scale = 1.0 / math.sqrt(DH)
    for g in range(G):
        qd, qv = _bf(torch, r.normal(size=(B * S, 3 * d)) * 1.5)
        dod, dov = _bf(torch, r.normal(size=(B * S, d)))
        qkvs.append(qd), douts.append(dod)
        os_.append(torch.zeros((B * S, d), dtype=torch.bfloat16, device="cuda"))
        lses.append(torch.zeros(B * H * S, device="cuda")), deltas.append(torch.zeros(B * H * S, device="cuda"))
        dqkvs.append(torch.full((B * S, 3 * d), 9.0, dtype=torch.bfloat16, device="cuda"))
        t = qv.reshape(B, S, 3, H, DH)
        q, k, v = (t[:, :, i].transpose(0, 2, 1, 3) for i in range(3))           # [B,H,S,DH]
        o, P = OL.attention_fwd(q, k, v, causal)
        do = dov.reshape(B, S, H, DH).transpose(0, 2, 1, 3)
        dq, dk, dv = OL.attention_bwd(q, k, v, P, do)
        sc = np.matmul(q, np.swapaxes(k, -1, -2)) * scale
        if causal:
            sc = np.where(np.tril(np.ones((S, S), dtype=bool)), sc, -np.inf)
        lse = np.log(np.exp(sc - sc.max(-1, keepdims=True)).sum(-1)) + sc.max(-1)
        refs.append((o, lse, dq, dk, dv))
    ops.hydra_op_attention_fwd(B, S, H, DH, 3 * d, d, causal, scale, qkvs, os_, lses)
    # the backward kernels read the forward's own (rounded) output, as they do in training
    ops.hydra_op_attention_bwd(B, S, H, DH, 3 * d, d, causal, scale, qkvs, os_, douts, lses, deltas, dqkvs)
    torch.cuda.synchronize()
    for g in range(G):
        o, lse, dq, dk, dv = refs[g]
        got_o = os_[g].double().cpu().numpy().reshape(B, S, H, DH).transpose(0, 2, 1, 3)
        # P is rounded to bf16 before P.v: error <= 2^-8 * sum_j P_ij |v_j| <= 2^-8 * max|v|; plus output rounding
        assert np.abs(got_o - o).max() <= 2.0 ** -7 * 8.0, f"o: {np.abs(got_o - o).max()}"
        assert np.sqrt(((got_o - o) ** 2).mean()) <= 4e-3 * np.sqrt((o ** 2).mean()), "o rms"
        assert np.allclose(lses[g].cpu().numpy().reshape(B, H, S), lse, rtol=1e-5, atol=1e-4)
        got = dqkvs[g].double().cpu().numpy().reshape(B, S, 3, H, DH)
        for name, i, ref in (("dq", 0, dq), ("dk", 1, dk), ("dv", 2, dv)):
            a = got[:, :, i].transpose(0, 2, 1, 3)
            rel = np.sqrt(((a - ref) ** 2).mean()) / np.sqrt((ref ** 2).mean())
            assert rel <= 1.5e-2, f"{name}: rel rms {rel}"
            assert np.abs(a - ref).max() <= 0.06 * np.abs(ref).max() + 1e-3, f"{name}: max {np.abs(a - ref).max()}"


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("shape", [(2, 64, 2, 64), (1, 80, 3, 64), (2, 200, 1, 64), (1, 512, 2, 64), (1, 136, 2, 128),
                                   (1, 33, 1, 128)])
def test_attention_forward_and_backward(torch, ops, causal, shape):
    B, S, H, DH = shape
    _attention_case(torch, ops, B, S, H, DH, causal, seed=S * DH + int(causal))


@pytest.mark.parametrize("shape", [(32, 512, 12, 64, False), (2, 2048, 8, 128, True)])
def test_attention_at_the_workloads_shapes(torch, ops, shape):
    """The attention of workload 2 at its full per-model size (batch 32, 12 heads of 64, S = 512: 8 key tiles per
    query block, 384 x 4 workgroups per problem, two problems grouped) and of workload 4's decoders (S = 2048, heads
    of 128, causal: 32 key tiles, short and long causal blocks dealt over the XCDs), the latter on 2 sequences x 8
    heads instead of 8 x 32 so that the fp64 oracle's probability matrices fit a test."""
    B, S, H, DH, causal = shape
    _attention_case(torch, ops, B, S, H, DH, causal, seed=S + DH)


@pytest.mark.parametrize("causal", [False, True])
def test_attention_over_128_key_tiles(torch, ops, causal):
    """One head of 64 at S = 8192 (the longest sequence the kernel rates are quoted at): the running maximum and sum go
    through 128 key tiles per query block, the backward kernels through 128 query tiles per key block."""
    _attention_case(torch, ops, 1, 8192, 1, 64, causal, seed=8192 + int(causal))


def test_attention_uniform_scores_closed_form(torch, ops):
    """q = k = 0 gives uniform probabilities: o is the running (causal) or global mean of v; lse = log(count)."""
    B, S, H, DH = 1, 96, 1, 64
    r = np.random.default_rng(0)
    qkv = np.zeros((S, 3 * DH))
    qkv[:, 2 * DH:] = r.normal(size=(S, DH))
    qd, qv = _bf(torch, qkv)
    for causal in (False, True):
        o = torch.zeros((S, DH), dtype=torch.bfloat16, device="cuda")
        lse = torch.zeros(S, device="cuda")
        ops.hydra_op_attention_fwd(B, S, H, DH, 3 * DH, DH, causal, 0.125, [qd], [o], [lse])
        torch.cuda.synchronize()
        v = qv[:, 2 * DH:]
        want = np.cumsum(v, 0) / np.arange(1, S + 1)[:, None] if causal else np.broadcast_to(v.mean(0), (S, DH))
        cnt = np.arange(1, S + 1) if causal else np.full(S, S)
        assert np.abs(o.double().cpu().numpy() - want).max() <= 2.0 ** -7 * np.abs(v).max()
        assert np.allclose(lse.cpu().numpy(), np.log(cnt), atol=1e-5)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("d,B,often", [(72, 3, 5), (328, 8, 16), (328, 9, 17), (256, 17, 19), (520, 16, 33), (264, 1, 4)])
def test_embedding_forward_and_backward(torch, ops, dtype, d, B, often):
    """One id that `often` tokens have (16 are added at a time, what is left in fours), rows wider than the 256 columns of a workgroup, batches
    of eight (a position's rows are added eight at a time) and what is left of them, positions past the sequence."""
    r = np.random.default_rng(5)
    V, S_table, S = 50, 40, 33
    mk = _bf if dtype else _f32
    ids = r.integers(0, V, size=(B, S)).astype(np.int32)
    ids[ids == 7] = 8
    ids.reshape(-1)[r.choice(B * S, size=often, replace=False)] = 7
    order = np.argsort(ids.reshape(-1), kind="stable").astype(np.int32)
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(ids.reshape(-1), minlength=V))]).astype(np.int32)
    toks, poss, xs, dxs, dtoks, dposs, refs = [], [], [], [], [], [], []
    for g in range(2):
        td, tv = mk(torch, r.normal(size=(V, d)))
        pd, pv = mk(torch, r.normal(size=(S_table, d)))
        dd, dv = mk(torch, r.normal(size=(B * S, d)))
        toks.append(td), poss.append(pd), dxs.append(dd)
        xs.append(torch.zeros((B * S, d), dtype=td.dtype, device="cuda"))
        dtoks.append(torch.full((V, d), 3.0, device="cuda")), dposs.append(torch.full((S_table, d), 3.0, device="cuda"))
        x = OL.embed_fwd(ids, tv, pv)
        dtok, dpos = OL.embed_bwd(ids, dv.reshape(B, S, d), V, S_table)
        refs.append((x, dtok, dpos))
    idd = torch.from_numpy(ids.reshape(-1)).cuda()
    ops.hydra_op_embed_fwd(dtype, B * S, S, d, d, idd, toks, poss, xs)
    ops.hydra_op_embed_bwd(dtype, V, S, S_table, B, d, d, torch.from_numpy(row_ptr).cuda(), torch.from_numpy(order).cuda(),
                           dxs, dtoks, dposs)
    torch.cuda.synchronize()
    for g in range(2):
        x, dtok, dpos = refs[g]
        tol = 2.0 ** -8 if dtype else 1e-6
        assert np.all(np.abs(xs[g].double().cpu().numpy().reshape(B, S, d) - x) <= tol * np.abs(x) + 1e-7)
        assert np.allclose(dtoks[g].cpu().numpy(), dtok, rtol=1e-5, atol=1e-5)
        assert np.allclose(dposs[g].cpu().numpy(), dpos, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("G,rows,d", [(2, 63, 512), (2, 129, 520), (1, 64, 8), (3, 65, 1024), (1, 1, 504), (4, 8193, 128), (16, 2051, 1016), (2, 1281, 264),
                                       (2, 1280, 1024), (3, 257, 40), (1, 4097, 616), (2, 4096, 640)])
def test_layernorm_row_batches(torch, ops, dtype, G, rows, d):
    """Row counts around a workgroup's 64 rows and a wave's batch, widths around the 512- and 1024-column limits, and launches large
    enough for several rows per wave in the forward pass, against fp64 (the column sums to 1e-5 of their terms' size)."""
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(rows * 31 + d)
    mk = lambda *sh: torch.randn(*sh, generator=gen, device="cuda")  # noqa: E731
    x, dy, add = ([mk(rows, d).to(t) for _ in range(G)] for _ in range(3))
    gamma, beta = [1 + 0.1 * mk(d) for _ in range(G)], [0.1 * mk(d) for _ in range(G)]
    y, dx = ([torch.zeros_like(u) for u in x] for _ in range(2))
    mean, rstd = ([torch.zeros(rows, device="cuda") for _ in range(G)] for _ in range(2))
    dg, db = ([torch.zeros(d, device="cuda") for _ in range(G)] for _ in range(2))
    part = [torch.zeros(ops.hydra_op_layernorm_part_floats(rows, d), device="cuda") for _ in range(G)]
    D = ops.BF16 if dtype == "bf16" else ops.F32
    ops.hydra_op_layernorm_fwd(D, rows, d, d, 1e-5, x, y, gamma, beta, mean, rstd)
    ops.hydra_op_layernorm_bwd(D, rows, d, d, x, dy, add, dx, gamma, mean, rstd, part, dg, db)
    tol = 2.0 ** -8 if dtype == "bf16" else 2e-6
    for g in range(G):
        xd, dyd = x[g].double(), dy[g].double()
        mu = xd.mean(1, keepdim=True)
        rs = ((xd - mu).square().mean(1, keepdim=True) + 1e-5).rsqrt()
        xh, gg = (xd - mu) * rs, dyd * gamma[g].double()
        want_y = xh * gamma[g].double() + beta[g].double()
        want_dx = rs * (gg - gg.mean(1, keepdim=True) - xh * (gg * xh).mean(1, keepdim=True)) + add[g].double()
        for got, want in ((y[g], want_y), (dx[g], want_dx)):
            err = (got.double() - want).abs()
            assert (err <= tol * (want.abs() + want.abs().mean())).all(), err.max()
        for got, term in ((dg[g], dyd * xh), (db[g], dyd)):
            assert ((got.double() - term.sum(0)).abs() <= 1e-5 * term.abs().sum(0) + 1e-6).all()


@pytest.mark.parametrize("DH,causal", [(64, False), (64, True), (128, False), (128, True)])
@pytest.mark.parametrize("S", [1, 63, 64, 65, 128, 200, 257])
def test_attention_reads_nothing_past_its_sequence(torch, ops, S, DH, causal):
    """Tiles of 64 rows go into LDS by loads that return zero past the sequence: with NaN in the sequence behind it every result of
    the first one keeps its bits, for odd and even numbers of tiles and partly filled ones; and it matches fp64 (bf16 rounding of
    the probabilities and of the results: 2^-7 of a row's largest terms)."""
    H, B, d = 2, 2, 2 * DH
    gen = torch.Generator(device="cuda").manual_seed(S * 3 + DH)
    t = B * S
    qkv0 = torch.randn(t, 3 * d, generator=gen, device="cuda").to(torch.bfloat16)
    do0 = torch.randn(t, d, generator=gen, device="cuda").to(torch.bfloat16)
    got = []
    for fill in (0.0, float("nan")):
        qkv, do = qkv0.clone(), do0.clone()
        qkv[S:], do[S:] = fill, fill
        o, dqkv = torch.zeros_like(do), torch.zeros_like(qkv)
        lse, delta = torch.zeros(t * H, device="cuda"), torch.zeros(t * H, device="cuda")
        ops.hydra_op_attention_fwd(B, S, H, DH, 3 * d, d, causal, DH ** -0.5, [qkv], [o], [lse])
        ops.hydra_op_attention_bwd(B, S, H, DH, 3 * d, d, causal, DH ** -0.5, [qkv], [o], [do], [lse], [delta], [dqkv])
        got.append((o[:S].clone(), lse[:H * S].clone(), dqkv[:S].clone()))
    assert all(torch.equal(a, b) for a, b in zip(*got))
    o, lse, dqkv = got[0]
    mask = torch.ones(S, S, device="cuda", dtype=torch.bool).triu(1)
    for h in range(H):
        q, k, v = (qkv0[:S, j * d + h * DH:j * d + (h + 1) * DH].double().contiguous() for j in range(3))
        dh = do0[:S, h * DH:(h + 1) * DH].double().contiguous()
        z = torch.mm(q, k.t().contiguous()) * DH ** -0.5
        if causal:
            z = z.masked_fill(mask, float("-inf"))
        ls = torch.logsumexp(z, 1)
        p = torch.exp(z - ls[:, None])
        oh = torch.mm(p, v)
        ds = p * (torch.mm(dh, v.t().contiguous()) - (dh * oh).sum(1, keepdim=True)) * DH ** -0.5
        want = (oh, torch.mm(ds, k), torch.mm(ds.t().contiguous(), q), torch.mm(p.t().contiguous(), dh))
        have = [o[:, h * DH:(h + 1) * DH]] + [dqkv[:, j * d + h * DH:j * d + (h + 1) * DH] for j in range(3)]
        for a, b in zip(have, want):
            assert (a.double() - b).abs().max() <= 2.0 ** -7 * max(float(b.abs().max()), 1.0)
        assert (lse[h * S:(h + 1) * S].double() - ls).abs().max() <= 1e-5


@pytest.mark.parametrize("S,H,DH,ld", [(3, 1, 64, 2 ** 27), (3, 1, 128, 2 ** 27), (5, 1, 64, 2 ** 26 + 8), (1, 2, 128, 2 ** 28), (3, 257, 64, 2 ** 27), (5, 2, 64, 2 ** 25 - 8),
                                       (3, 161, 128, 2 ** 27)])
def test_attention_rows_of_a_short_sequence_far_apart(torch, ops, S, H, DH, ld):
    """Rows of some hundred megabytes: offsets of a block's rows past the sequence would come round to rows that are there.  The bits of packed matrices,
    and nothing but the heads' own columns is written, against both halves of the backward pass in one launch and in two."""
    d, gen = H * DH, torch.Generator(device="cuda").manual_seed(S + DH)
    qkv0, do0 = (torch.randn(S, n, generator=gen, device="cuda").to(torch.bfloat16) for n in (3 * d, d))
    got = []
    for far in (False, True):
        lq, lo = (ld, ld) if far else (3 * d, d)
        qkv, dqkv, o, do = (torch.full((S, n), float("nan"), device="cuda", dtype=torch.bfloat16) for n in (lq, lq, lo, lo))
        qkv[:, :3 * d], do[:, :d] = qkv0, do0
        lse, delta = torch.zeros(S * H, device="cuda"), torch.zeros(S * H, device="cuda")
        ops.hydra_op_attention_fwd(1, S, H, DH, lq, lo, True, DH ** -0.5, [qkv], [o], [lse])
        ops.hydra_op_attention_bwd(1, S, H, DH, lq, lo, True, DH ** -0.5, [qkv], [o], [do], [lse], [delta], [dqkv])
        assert torch.isnan(o[:, d:]).all() and torch.isnan(dqkv[:, 3 * d:]).all()
        got.append((o[:, :d].clone(), dqkv[:, :3 * d].clone(), lse, delta))
        assert all(torch.isfinite(x).all() for x in got[-1])
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("B,S,H,DH,causal", [(1, 200, 2, 64, False), (2, 77, 3, 64, True), (1, 300, 2, 128, True), (3, 64, 1, 128, False)])
def test_attention_backward_in_one_launch_equals_two(torch, ops, B, S, H, DH, causal):
    """Small launches run both halves of the backward pass as one kernel; the same problem in a group too large for that must give
    the same bits, delta included."""
    d, t = H * DH, B * S
    gen = torch.Generator(device="cuda").manual_seed(S + DH)
    qkv = torch.randn(t, 3 * d, generator=gen, device="cuda").to(torch.bfloat16)
    do = torch.randn(t, d, generator=gen, device="cuda").to(torch.bfloat16)
    per = (S + 127) // 128 * B * H
    for rep in (1, 256 // per + 1):  # copies of the batch: the second is past 256 row blocks
        n = rep * B
        q, g = qkv.repeat(rep, 1), do.repeat(rep, 1)
        o, dqkv = torch.zeros_like(g), torch.zeros_like(q)
        lse, delta = torch.zeros(rep * t * H, device="cuda"), torch.zeros(rep * t * H, device="cuda")
        ops.hydra_op_attention_fwd(n, S, H, DH, 3 * d, d, causal, DH ** -0.5, [q], [o], [lse])
        ops.hydra_op_attention_bwd(n, S, H, DH, 3 * d, d, causal, DH ** -0.5, [q], [o], [g], [lse], [delta], [dqkv])
        if rep == 1:
            first = dqkv.clone(), delta.clone()
    assert torch.equal(dqkv[:t], first[0]) and torch.equal(dqkv[-t:], first[0])
    assert torch.equal(delta[:t * H], first[1])


@pytest.mark.parametrize("B,S,H,DH", [(53, 449, 5, 64), (33, 512, 5, 128), (9, 1000, 5, 64), (9, 1024, 5, 128), (6, 1410, 10, 128), (41, 700, 5, 64),
                                      (3, 1985, 7, 64), (2, 2048, 9, 128)])
def test_causal_attention_in_pairs_of_row_blocks_equals_single_ones(torch, ops, B, S, H, DH):
    """Large causal launches give a workgroup two row blocks of a head, one after the other; every batch row gives the bits it gives alone,
    in a launch too small for that, with a last block that is full or down to one row and odd and even numbers of tiles."""
    d, gen = H * DH, torch.Generator(device="cuda").manual_seed(S + DH)
    qkv = torch.randn(B * S, 3 * d, generator=gen, device="cuda").to(torch.bfloat16)
    do = torch.randn(B * S, d, generator=gen, device="cuda").to(torch.bfloat16)

    def both(n, q, g):
        o, dqkv = torch.zeros_like(g), torch.zeros_like(q)
        lse, delta = (torch.zeros(n * S * H, device="cuda") for _ in range(2))
        ops.hydra_op_attention_fwd(n, S, H, DH, 3 * d, d, True, DH ** -0.5, [q], [o], [lse])
        ops.hydra_op_attention_bwd(n, S, H, DH, 3 * d, d, True, DH ** -0.5, [q], [o], [g], [lse], [delta], [dqkv])
        return o, dqkv, lse, delta

    whole = both(B, qkv, do)
    for b in range(B):
        rows = slice(b * S, (b + 1) * S)
        part = both(1, qkv[rows].clone(), do[rows].clone())
        for w, x in zip(whole, part):
            assert torch.equal(w[b * len(x):(b + 1) * len(x)], x)


@pytest.mark.parametrize("off", [1, 2, 4, 7])
def test_attention_writes_to_buffers_of_any_alignment(torch, ops, off):
    """o and dqkv need no alignment beyond an element's: the same bits, and nothing outside of them."""
    B, S, H, DH = 2, 150, 2, 64
    d, t, gen = H * DH, B * S, torch.Generator(device="cuda").manual_seed(off)
    qkv = torch.randn(t, 3 * d, generator=gen, device="cuda").to(torch.bfloat16)
    do = torch.randn(t, d, generator=gen, device="cuda").to(torch.bfloat16)
    got = []
    for k in (0, off):
        o_all, dq_all = (torch.full((n + 64,), 7.0, device="cuda", dtype=torch.bfloat16) for n in (t * d, 3 * t * d))
        o, dqkv = o_all[16 + k:16 + k + t * d].view(t, d), dq_all[16 + k:16 + k + 3 * t * d].view(t, 3 * d)
        lse, delta = (torch.zeros(t * H, device="cuda") for _ in range(2))
        ops.hydra_op_attention_fwd(B, S, H, DH, 3 * d, d, False, DH ** -0.5, [qkv], [o], [lse])
        ops.hydra_op_attention_bwd(B, S, H, DH, 3 * d, d, False, DH ** -0.5, [qkv], [o], [do], [lse], [delta], [dqkv])
        got.append((o.clone(), dqkv.clone()))
        for x, n in ((o_all, t * d), (dq_all, 3 * t * d)):
            assert bool((x[:16 + k] == 7.0).all()) and bool((x[16 + k + n:] == 7.0).all())
    assert all(torch.equal(a, b) for a, b in zip(*got))


def attention_bits(torch, ops, G, B, S, H, DH, causal):
    """Digest of o, lse, dqkv of G problems of frozen pseudo-random inputs."""
    d, t, r = H * DH, B * S, np.random.RandomState(S * 7 + DH)
    mk = lambda *sh: torch.from_numpy(r.standard_normal(sh).astype(np.float32)).to(torch.bfloat16).cuda()  # noqa: E731
    qkv, do = [mk(t, 3 * d) for _ in range(G)], [mk(t, d) for _ in range(G)]
    o, dqkv = [torch.zeros_like(x) for x in do], [torch.zeros_like(x) for x in qkv]
    lse, delta = ([torch.zeros(t * H, device="cuda") for _ in range(G)] for _ in range(2))
    ops.hydra_op_attention_fwd(B, S, H, DH, 3 * d, d, causal, DH ** -0.5, qkv, o, lse)
    ops.hydra_op_attention_bwd(B, S, H, DH, 3 * d, d, causal, DH ** -0.5, qkv, o, do, lse, delta, dqkv)
    h = hashlib.sha256()
    for x in o + lse + dqkv:
        h.update(x.cpu().view(torch.uint8).numpy().tobytes())
    return h.hexdigest()[:32]


def _golden_lines(name):
    with open(os.path.join(os.path.dirname(__file__), "golden", name)) as f:
        return [ln.split() for ln in f if ln.strip() and not ln.startswith("#")]


@pytest.mark.parametrize("line", _golden_lines("attention_bits.txt"), ids=lambda ln: "x".join(ln[:6]))
def test_attention_keeps_its_bits(torch, ops, line):
    """A training run repeats itself bit for bit from one version of the kernels to the next: the order of the row sums, of dO.O and of
    dP - delta is part of the result (twenty Adam steps turn a changed last bit into 1e-3 of a parameter)."""
    assert attention_bits(torch, ops, *[int(x) for x in line[:6]]) == line[6]


@pytest.mark.parametrize("G,B,S,H,DH,causal", [(1, 1, 1, 1, 64, False), (3, 2, 129, 1, 64, True), (2, 3, 127, 5, 128, False), (2, 5, 257, 3, 64, False),
                                                (5, 7, 300, 7, 64, True), (1, 2, 385, 3, 128, True)])
def test_attention_of_a_group_equals_its_parts(torch, ops, G, B, S, H, DH, causal):
    """A workgroup finds its problem, batch row, head and row block by multiplications with reciprocals: every (problem, batch row) of a
    launch gives the bits it gives alone, at counts of one and at ones that divide nothing."""
    d, gen = H * DH, torch.Generator(device="cuda").manual_seed(S * 31 + H)
    mk = lambda n: torch.randn(n, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    qkv, do = [mk(B * S * 3 * d).view(B * S, 3 * d) for _ in range(G)], [mk(B * S * d).view(B * S, d) for _ in range(G)]

    def run(qs, gs, b):
        o, dq = [torch.full_like(x, 7.0) for x in gs], [torch.full_like(x, 7.0) for x in qs]
        lse, delta = ([torch.full((b * H * S,), 7.0, device="cuda") for _ in qs] for _ in range(2))
        ops.hydra_op_attention_fwd(b, S, H, DH, 3 * d, d, causal, DH ** -0.5, qs, o, lse)
        ops.hydra_op_attention_bwd(b, S, H, DH, 3 * d, d, causal, DH ** -0.5, qs, o, gs, lse, delta, dq)
        return o, lse, delta, dq

    whole = run(qkv, do, B)
    for g in range(G):
        for b in range(B):
            r, hs = slice(b * S, (b + 1) * S), slice(b * H * S, (b + 1) * H * S)
            part = run([qkv[g][r].contiguous()], [do[g][r].contiguous()], 1)
            for w, p, sl in zip(whole, part, (r, hs, hs, r)):
                assert torch.equal(w[g][sl], p[0]), (g, b)


def _column_sums(dv, xh, rows):
    """dgamma, dbeta in fp32 in the order the kernels add them: rows r, r + 4, ... of a block of 64 are a chain of fused multiply-adds,
    four chains make the block's partial sum, the blocks are added in 16 ranges.  (64-bit mantissas hold the products; the fused
    rounding is taken from them.)"""
    nb, d = -(-rows // 64), dv.shape[1]
    f, pad = np.float32, lambda a: np.concatenate([a, np.zeros((nb * 64 - rows, d), np.float32)]).reshape(nb, 16, 4, d)  # noqa: E731
    v, h = pad(dv), pad(xh)
    sg, sb = np.zeros((nb, 4, d), f), np.zeros((nb, 4, d), f)
    for i in range(16):
        sg = (v[:, i].astype(np.longdouble) * h[:, i] + sg).astype(f)
        sb = sb + v[:, i]
    per, out = (nb + 15) // 16, []
    for chains in (sg, sb):
        part, s = np.zeros((nb, d), f), np.zeros(d, f)
        for w in range(4):
            part = part + chains[:, w]
        for w in range(16):
            t = np.zeros(d, f)
            for b in range(w * per, min(nb, (w + 1) * per)):
                t = t + part[b]
            s = s + t
        out.append(s)
    return out


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("G,rows,d", [(1, 1, 8), (2, 67, 64), (4, 1024, 256), (1, 1100, 200), (1, 1280, 512), (1, 1281, 264), (1, 2000, 768), (3, 1000, 1000),
                                       (2, 2100, 512), (4, 6000, 40), (1, 16500, 160), (1, 16500, 512), (2, 5300, 1000), (1, 1024, 1024)])
def test_layernorm_column_sums_keep_their_order(torch, ops, dtype, G, rows, d):
    """Every kernel the backward pass may take (one launch or two, few rows or many) adds dgamma and dbeta in one order, which is part of
    the result: the sums of the first and last problem bit for bit."""
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(rows + d)
    mk = lambda *sh: torch.randn(*sh, generator=gen, device="cuda")  # noqa: E731
    x, dy = ([mk(rows, d).to(t) for _ in range(G)] for _ in range(2))
    gamma, beta = [1 + 0.1 * mk(d) for _ in range(G)], [0.1 * mk(d) for _ in range(G)]
    y, dx = ([torch.zeros_like(u) for u in x] for _ in range(2))
    mean, rstd = ([torch.zeros(rows, device="cuda") for _ in range(G)] for _ in range(2))
    dg, db = ([torch.zeros(d, device="cuda") for _ in range(G)] for _ in range(2))
    part = [torch.zeros(ops.hydra_op_layernorm_part_floats(rows, d), device="cuda") for _ in range(G)]
    D = ops.BF16 if dtype == "bf16" else ops.F32
    ops.hydra_op_layernorm_fwd(D, rows, d, d, 1e-5, x, y, gamma, beta, mean, rstd)
    ops.hydra_op_layernorm_bwd(D, rows, d, d, x, dy, None, dx, gamma, mean, rstd, part, dg, db)
    for g in {0, G - 1}:
        dv = dy[g].float().cpu().numpy()
        xh = (x[g].float() - mean[g][:, None]) * rstd[g][:, None]
        want = _column_sums(dv, xh.cpu().numpy(), rows)
        for got, w in zip((dg[g], db[g]), want):
            assert np.array_equal(got.cpu().numpy(), w)


@pytest.mark.parametrize("G,rows,d", [(3, 16500, 520), (4, 12321, 1024), (7, 7041, 1000)])
def test_layernorm_column_sums_with_four_workgroups_to_a_cu(torch, ops, G, rows, d):
    """More than three blocks of 64 rows per compute unit, rows wider than 512: the kernel that reads gamma from LDS keeps the order, too."""
    test_layernorm_column_sums_keep_their_order(torch, ops, "bf16", G, rows, d)


@pytest.mark.parametrize("over", ["x", "dy", "add"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("G,rows,d", [(2, 256, 256), (1, 1200, 1000), (1, 2000, 768), (2, 5000, 512), (3, 90, 1536)])
def test_layernorm_backward_in_place(torch, ops, dtype, over, G, rows, d):
    """dx written over x, dy or the additive term: the bits of the same call with a buffer of its own (column sums included: they are
    made from x and dy, which the rows' own pass is overwriting)."""
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(rows + d)
    mk = lambda *sh: torch.randn(*sh, generator=gen, device="cuda")  # noqa: E731
    src = {n: [mk(rows, d).to(t) for _ in range(G)] for n in ("x", "dy", "add")}
    gamma = [1 + 0.1 * mk(d) for _ in range(G)]
    mean, rstd = [u.float().mean(1) for u in src["x"]], [u.float().var(1, unbiased=False).add(1e-5).rsqrt() for u in src["x"]]
    got = []
    for in_place in (False, True):
        s = {n: [u.clone() for u in us] for n, us in src.items()}
        dx = s[over] if in_place else [torch.zeros_like(u) for u in s["x"]]
        dg, db = ([torch.zeros(d, device="cuda") for _ in range(G)] for _ in range(2))
        part = [torch.zeros(ops.hydra_op_layernorm_part_floats(rows, d), device="cuda") for _ in range(G)]
        ops.hydra_op_layernorm_bwd(ops.BF16 if dtype == "bf16" else ops.F32, rows, d, d, s["x"], s["dy"], s["add"], dx, gamma, mean, rstd,
                                   part, dg, db)
        got.append(dx + dg + db)
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("with_add", [True, False])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,d,ld", [(16449, 184, 192), (16449, 512, 512), (16449, 520, 1040), (57345, 776, 776), (16449, 1016, 1024), (16449, 1800, 1800),
                                       (22529, 2048, 2048), (99, 1032, 1040), (4129, 2056, 2064)])
def test_layernorm_backward_from_any_address(torch, ops, dtype, with_add, rows, d, ld):
    """Matrices that start one element behind a 16-byte boundary (bf16: half a word, through the same descriptors) give the bits of matrices that
    start on one, a third of the rows, which may be another kernel's, has the same dx, the last block of rows holds few of them, and what lies
    behind a row's end is not written."""
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(rows + d)
    src = [torch.randn(rows, ld, generator=gen, device="cuda").to(t) for _ in range(3)]
    gamma = [1 + 0.1 * torch.randn(d, generator=gen, device="cuda")]
    v = src[0][:, :d].float()
    mean, rstd = [v.mean(1)], [v.var(1, unbiased=False).add(1e-5).rsqrt()]
    got = []
    for shift, n in ((0, rows), (1, rows), (0, rows // 3)):
        x, dy, add, dx = (torch.full((rows * ld + 8,), 7.0, device="cuda", dtype=t)[shift:shift + rows * ld].view(rows, ld) for _ in range(4))
        for to, of in zip((x, dy, add), src):
            to.copy_(of)
        dg, db = torch.zeros(d, device="cuda"), torch.zeros(d, device="cuda")
        part = [torch.zeros(ops.hydra_op_layernorm_part_floats(rows, d), device="cuda")]
        ops.hydra_op_layernorm_bwd(ops.BF16 if dtype == "bf16" else ops.F32, n, d, ld, [x], [dy], [add] if with_add else None, [dx], gamma,
                                   mean, rstd, part, [dg], [db])
        assert bool((dx[:, d:] == 7.0).all()) and bool((dx[n:] == 7.0).all())
        got.append((dx[:, :d].clone(), dg, db))
    assert all(torch.equal(a, b) for a, b in zip(*got[:2]))
    assert torch.equal(got[0][0][:rows // 3], got[2][0][:rows // 3])


@pytest.mark.parametrize("with_add", [True, False])
@pytest.mark.parametrize("rows,d", [(8225, 1544), (8500, 2048), (10209, 2040)])
def test_layernorm_backward_bits_do_not_depend_on_the_group(torch, ops, with_add, rows, d):
    """fp32 rows of 1544 to 2048 elements: two problems in 513 to 640 row blocks take the kernel without look-ahead, each of them alone the one with
    it; dx, dgamma and dbeta are the same bits."""
    gen = torch.Generator(device="cuda").manual_seed(rows + d)
    x, dy, add = ([torch.randn(rows, d, generator=gen, device="cuda") for _ in range(2)] for _ in range(3))
    gamma = [1 + 0.1 * torch.randn(d, generator=gen, device="cuda") for _ in range(2)]
    mean, rstd = [v.mean(1) for v in x], [v.var(1, unbiased=False).add(1e-5).rsqrt() for v in x]

    def run(which):
        pick = lambda ts: [ts[i] for i in which]  # noqa: E731
        dx, (dg, db) = [torch.zeros(rows, d, device="cuda") for _ in which], ([torch.zeros(d, device="cuda") for _ in which] for _ in range(2))
        part = [torch.zeros(ops.hydra_op_layernorm_part_floats(rows, d), device="cuda") for _ in which]
        ops.hydra_op_layernorm_bwd(ops.F32, rows, d, d, pick(x), pick(dy), pick(add) if with_add else None, dx, pick(gamma), pick(mean), pick(rstd),
                                   part, dg, db)
        return list(zip(dx, dg, db))

    together = run((0, 1))
    for i in (0, 1):
        for a, b in zip(together[i], run((i,))[0]):
            assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,d", [(8195, 256), (8193, 904), (8194, 1024)])
def test_layernorm_forward_bits_do_not_depend_on_the_group(torch, ops, dtype, rows, d):
    """A group of four is large enough for several rows per wave, one problem alone is not: the same bits."""
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(rows + d)
    mk = lambda *sh: torch.randn(*sh, generator=gen, device="cuda")  # noqa: E731
    x, gamma, beta = [mk(rows, d).to(t) for _ in range(4)], [1 + 0.1 * mk(d) for _ in range(4)], [0.1 * mk(d) for _ in range(4)]
    got = []
    for n in (4, 1):
        y = [torch.zeros_like(u) for u in x[:n]]
        mean, rstd = ([torch.zeros(rows, device="cuda") for _ in range(n)] for _ in range(2))
        ops.hydra_op_layernorm_fwd(ops.BF16 if dtype == "bf16" else ops.F32, rows, d, d, 1e-5, x[:n], y, gamma[:n], beta[:n], mean, rstd)
        got.append((y[0], mean[0], rstd[0]))
    assert all(torch.equal(a, b) for a, b in zip(*got))


def test_attention_refuses_tiles_it_cannot_load(torch, ops):
    """The matrices whose tiles are loaded straight into LDS must start on 16 bytes, and 64 of their rows must lie within 2 GiB: an
    argument error, not a launch, otherwise."""
    S, H, DH = 64, 2, 64
    d = H * DH
    mk = lambda n, off: torch.zeros(S * n + 8, device="cuda", dtype=torch.bfloat16)[off:off + S * n].view(S, n)  # noqa: E731
    o, lse, delta, dqkv = mk(d, 0), torch.zeros(S * H, device="cuda"), torch.zeros(S * H, device="cuda"), mk(3 * d, 0)
    fwd = lambda q: ops.hydra_op_attention_fwd(1, S, H, DH, 3 * d, d, False, 0.125, [q], [o], [lse])  # noqa: E731
    bwd = lambda q, g: ops.hydra_op_attention_bwd(1, S, H, DH, 3 * d, d, False, 0.125, [q], [o], [g], [lse], [delta], [dqkv])  # noqa: E731
    fwd(mk(3 * d, 0)), bwd(mk(3 * d, 0), mk(d, 0))
    far = lambda: ops.hydra_op_attention_fwd(1, S, H, DH, 1 << 24, d, False, 0.125, [mk(3 * d, 0)], [o], [lse])  # noqa: E731
    for call in (far, lambda: fwd(mk(3 * d, 4)), lambda: bwd(mk(3 * d, 4), mk(d, 0)), lambda: bwd(mk(3 * d, 0), mk(d, 4))):
        with pytest.raises(Exception, match="attention"):
            call()


@pytest.mark.parametrize("B,S,H,DH,causal", [(2, 200, 2, 64, False), (1, 300, 2, 128, True), (8, 512, 16, 64, False)])
def test_attention_backward_over_its_output(torch, ops, B, S, H, DH, causal):
    """o kept in the query columns of the buffer that dqkv overwrites: the bits of the same call with a buffer of its own, for few row
    blocks and many."""
    d, t = H * DH, B * S
    gen = torch.Generator(device="cuda").manual_seed(S)
    qkv, do = (torch.randn(t, n * d, generator=gen, device="cuda").to(torch.bfloat16) for n in (3, 1))
    do3, got = torch.zeros_like(qkv), []
    do3[:, :d] = do
    for own in (True, False):
        o, dqkv = torch.zeros_like(qkv), torch.zeros_like(qkv)
        lse, delta = torch.zeros(t * H, device="cuda"), torch.zeros(t * H, device="cuda")
        ops.hydra_op_attention_fwd(B, S, H, DH, 3 * d, 3 * d, causal, DH ** -0.5, [qkv], [o], [lse])
        dst = dqkv if own else o
        ops.hydra_op_attention_bwd(B, S, H, DH, 3 * d, 3 * d, causal, DH ** -0.5, [qkv], [o], [do3], [lse], [delta], [dst])
        got.append((dst, delta))
    assert all(torch.equal(a, b) for a, b in zip(*got))
