"""GPU parity: tree-correct causal convolution (forward and backward) against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2511_00413_amd as T
import workloads as W
from oracle import meta as M
from oracle import ssm as S
from tt_testutil import rel_l2

pytestmark = pytest.mark.gpu


def _inputs(n, c, k, seed, dtype):
    g = torch.Generator().manual_seed(seed)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn((n, c), generator=g).to(tdt)
    dy = torch.randn((n, c), generator=g).to(tdt)
    w = torch.randn((c, k), generator=g) * 0.5
    b = torch.randn(c, generator=g) * 0.1
    return x, dy, w, b


def _run_and_check(tok_pred, n, c, k, seed, dtype, silu=True, bias=True):
    x, dy, w, b = _inputs(n, c, k, seed, dtype)
    if not bias:
        b = None
    act = "silu" if silu else None
    want_y, _ = S.tree_conv(x, w, b, tok_pred, act)
    want_dx, want_dw, want_db = S.tree_conv_bwd(x, w, b, tok_pred, dy, act)
    pred_d = torch.from_numpy(np.asarray(tok_pred, dtype=np.int32)).cuda()
    xd, dyd, wd, bd = x.cuda(), dy.cuda(), w.cuda(), None if b is None else b.cuda()
    plan = T.tree_conv_plan(tok_pred, k)
    print(f"[case] tree conv n={n} C={c} K={k} {dtype} silu={silu} bias={bias}: {len(plan.fix_tok)} fix-up tokens", flush=True)
    y = T.tree_conv_fwd(xd, wd, bd, pred_d, silu=silu)
    dx, dw, db = T.tree_conv_bwd(xd, wd, bd, pred_d, dyd, plan, silu=silu, want_dbias=bias)
    torch.cuda.synchronize()
    tol = 4e-3 if dtype == "bf16" else 2e-6           # bf16: one rounding of the output (2^-9 relative)
    errs = dict(y=rel_l2(y.float().cpu().numpy(), want_y), dx=rel_l2(dx.float().cpu().numpy(), want_dx),
                dw=rel_l2(dw.cpu().numpy(), want_dw))
    if bias:
        errs["db"] = rel_l2(db.cpu().numpy(), want_db)
    print("   rel-L2:", {k_: f"{e:.2e}" for k_, e in errs.items()}, flush=True)
    assert errs["y"] <= tol and errs["dx"] <= tol
    assert errs["dw"] <= 1e-5 and errs.get("db", 0.0) <= 1e-5      # fp32 sums of exact products
    # element-wise on the fix-up rows and their neighbours (a wrong successor shows up there)
    rows = np.unique(np.clip(np.concatenate([plan.fix_tok, plan.fix_tok + 1, plan.fix_t, [0, n - 1]]), 0, n - 1))
    a, bq = dx.float().cpu().numpy()[rows], want_dx[rows]
    assert np.abs(a - bq).max() <= (3e-2 if dtype == "bf16" else 1e-4) * max(1.0, np.abs(bq).max())
    return y, dx, dw, db


@pytest.mark.parametrize("seed,k,dtype,c", [(0, 4, "bf16", 64), (1, 3, "bf16", 128), (2, 2, "fp32", 32), (3, 4, "fp32", 64),
                                             (4, 4, "bf16", 8), (5, 4, "fp32", 4)])
def test_random_trees_short_nodes(seed, k, dtype, c):
    """Nodes of 0..4 tokens: windows cross several nodes, branch points everywhere."""
    t = W.random_tree(950 + seed, n_nodes=40 + 10 * seed, lo=1, hi=4, n_roots=1 + seed % 2, p_zero=0.2)
    m = M.dfs_meta(t.parent, t.seg_len)
    _run_and_check(m["tok_pred"], m["n_tokens"], c, k, seed, dtype)


@pytest.mark.parametrize("nodes,hi,k,dtype,c", [(1, 31, 4, "bf16", 8), (20, 40, 4, "bf16", 24), (26, 40, 3, "fp32", 12),
                                                (30, 40, 2, "bf16", 8), (400, 3, 4, "bf16", 40), (90, 12, 3, "bf16", 16)])
def test_weight_gradient_segments_and_run_ends(nodes, hi, k, dtype, c):
    """Fewer tiles than the 16 segments of the weight-gradient sum, about as many and more; output counts that do not fill
    its workgroups; branch-point rows whose successors stop short (one-token children, the end of the sequence)."""
    t = W.random_tree(1200 + nodes, n_nodes=nodes, lo=1, hi=hi)
    m = M.dfs_meta(t.parent, t.seg_len)
    _run_and_check(m["tok_pred"], m["n_tokens"], c, k, nodes, dtype)


@pytest.mark.parametrize("silu,bias", [(False, True), (True, False), (False, False)])
def test_activation_and_bias_variants(silu, bias):
    t = W.random_tree(971, n_nodes=30, lo=1, hi=30)
    m = M.dfs_meta(t.parent, t.seg_len)
    _run_and_check(m["tok_pred"], m["n_tokens"], 128, 4, 7, "bf16", silu=silu, bias=bias)


def test_many_tiles_ragged_tail_and_reproducible():
    """Several thousand tokens (many token tiles, a ragged last one), a few hundred channels."""
    t = W.random_tree(981, n_nodes=60, lo=20, hi=200)
    m = M.dfs_meta(t.parent, t.seg_len)
    n = m["n_tokens"]
    assert n % 64 != 0
    y, dx, dw, db = _run_and_check(m["tok_pred"], n, 328, 4, 11, "bf16")
    y2, dx2, dw2, db2 = _run_and_check(m["tok_pred"], n, 328, 4, 11, "bf16")
    for a, b in ((y, y2), (dx, dx2), (dw, dw2), (db, db2)):
        assert torch.equal(a, b)


# Long tiles of the backward walk (the short ones of 32 tokens are what small shapes get): fp32 in one round of workgroups (tiles of
# 71 tokens), in one round of the longest tiles and beyond it in two (136), bf16 tiles of 94 and 188 tokens (no multiple of a batch) and of
# 256, every kernel size.
@pytest.mark.parametrize("n,c,k,dtype", [(9001, 4096, 3, "fp32"), (9001, 4096, 2, "fp32"), (17003, 4096, 4, "fp32"), (16800, 8192, 4, "fp32"),
                                         (17003, 8192, 3, "fp32"), (9001, 8192, 3, "bf16"), (18003, 8192, 4, "bf16"), (26001, 8192, 2, "bf16")])
def test_long_tiles(n, c, k, dtype):
    """The channels are independent: eight of them (the first and the last lanes of a row) against the oracle."""
    t = W.random_tree(990 + k, n_nodes=120, lo=1, hi=n // 50)
    seg = np.maximum(1, np.floor(np.asarray(t.seg_len) * (n / t.n_tokens))).astype(np.int32)
    seg[-1] += n - seg.sum()
    pred = M.dfs_meta(t.parent, seg)["tok_pred"]
    g = torch.Generator(device="cuda").manual_seed(n + c)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x, dy = (torch.randn((n, c), generator=g, device="cuda").to(tdt) for _ in range(2))
    w, b = torch.randn((c, k), generator=g, device="cuda") * 0.5, torch.randn(c, generator=g, device="cuda") * 0.1
    plan = T.tree_conv_plan(pred, k)
    print(f"[case] tree conv n={n} C={c} K={k} {dtype}, long tiles: {len(plan.fix_tok)} fix-up tokens", flush=True)
    pred_d = torch.from_numpy(pred).cuda()
    y = T.tree_conv_fwd(x, w, b, pred_d)
    dx, dw, db = T.tree_conv_bwd(x, w, b, pred_d, dy, plan)
    some = [0, 1, 2, 3, c - 4, c - 3, c - 2, c - 1]
    xs, dys, ws, bs = x[:, some].cpu(), dy[:, some].cpu(), w[some].cpu(), b[some].cpu()
    want_y, _ = S.tree_conv(xs, ws, bs, pred, "silu")
    want_dx, want_dw, want_db = S.tree_conv_bwd(xs, ws, bs, pred, dys, "silu")
    tol = 4e-3 if dtype == "bf16" else 2e-6           # bf16: one rounding of the output (2^-9 relative)
    got_dx = dx[:, some].float().cpu().numpy()
    assert rel_l2(y[:, some].float().cpu().numpy(), want_y) <= tol and rel_l2(got_dx, want_dx) <= tol
    assert np.abs(got_dx - want_dx).max() <= (3e-2 if dtype == "bf16" else 1e-4) * np.abs(want_dx).max()
    # fp32 sums, on 512 channels in float64 (the error of a few sums scatters): a chain of L additions of terms of either sign adds
    # about 2^-24 sqrt(0.085 L) of the sum: 2.8e-7 for a chain of 256 tokens; a chain of 24, one of the 11 chains of a tile, one of
    # the tiles and the last rounding 1.5e-7 together
    assert rel_l2(dw[some].cpu().numpy(), want_dw) <= 2e-5 and rel_l2(db[some].cpu().numpy(), want_db) <= 2e-5
    at = torch.arange(0, c, c // 512, device="cuda")
    xa = torch.cat([x[:, at].double(), torch.zeros((1, len(at)), dtype=torch.float64, device="cuda")])    # row -1: no predecessor
    back, taps = torch.arange(n, device="cuda"), []
    for _ in range(k):
        taps.insert(0, xa[back])
        back = torch.where(back >= 0, pred_d[back].long(), -1)
    z = b[at].double() + sum(w[at, j].double() * taps[j] for j in range(k))
    dz = dy[:, at].double() * torch.sigmoid(z) * (1 + z * (1 - torch.sigmoid(z)))
    exact_dw, exact_db = torch.stack([(dz * taps[j]).sum(0) for j in range(k)], dim=1), dz.sum(0)
    errs = [float((got.double() - want).norm() / want.norm()) for got, want in ((dw[at], exact_dw), (db[at], exact_db))]
    assert max(errs) <= 1.9e-7


def test_strided_rows_and_chain():
    """x and dy as column slices of wider buffers; a plain chain equals a library causal conv1d."""
    n, c, k = 700, 64, 4
    tok_pred = np.arange(-1, n - 1, dtype=np.int32)
    x, dy, w, b = _inputs(n, 2 * c, k, 3, "bf16")
    xs, dys = x.cuda()[:, c:], dy.cuda()[:, :c]
    w, b = w[:c].contiguous(), b[:c].contiguous()
    pred_d = torch.from_numpy(tok_pred).cuda()
    plan = T.tree_conv_plan(tok_pred, k)
    assert len(plan.fix_tok) == 0
    print("[case] tree conv strided rows, chain", flush=True)
    y = T.tree_conv_fwd(xs, w.cuda(), b.cuda(), pred_d)
    dx, dw, db = T.tree_conv_bwd(xs, w.cuda(), b.cuda(), pred_d, dys, plan)
    torch.cuda.synchronize()
    xt = x[:, c:].double().requires_grad_(True)
    wt, bt = w.double().requires_grad_(True), b.double().requires_grad_(True)
    z = torch.nn.functional.conv1d(torch.nn.functional.pad(xt.T[None], (k - 1, 0)), wt[:, None, :], bt, groups=c)[0].T
    ref = torch.nn.functional.silu(z)
    (ref * dy[:, :c].double()).sum().backward()
    assert rel_l2(y.float().cpu().numpy(), ref.detach().numpy()) <= 4e-3
    assert rel_l2(dx.float().cpu().numpy(), xt.grad.numpy()) <= 4e-3
    assert rel_l2(dw.cpu().numpy(), wt.grad.numpy()) <= 1e-5 and rel_l2(db.cpu().numpy(), bt.grad.numpy()) <= 1e-5


def test_errors():
    x = torch.zeros((8, 16), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((16, 5), dtype=torch.float32, device="cuda")
    pred = torch.arange(-1, 7, dtype=torch.int32, device="cuda")
    with pytest.raises(T.TreeTrainError) as e:
        T.tree_conv_fwd(x, w, None, pred)
    assert e.value.status == -8
    w = torch.zeros((12, 4), dtype=torch.float32, device="cuda")
    with pytest.raises(T.TreeTrainError) as e:
        T.tree_conv_fwd(x[:, :12], w, None, pred)
    assert e.value.status == -2
