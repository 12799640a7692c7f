"""GPU parity: backward of the gated delta rule with tree state routing against the fp64 reverse recurrence.
Like the forward, the kernels round the operands of their matrix products to bf16 once each (per-chunk
operands, entering state, R, Vn, gradient of the leaving state, dVn, dR) and accumulate in
fp32; the inverse of a chunk's triangular system and element-wise work are fp32; dq, dk, dv are rounded to bf16 at the end (dq, dk after the fp32 sum
over the value heads of a key head).  Tolerance: rel-L2 <= 8e-3 on every output (a product of two or three
operands rounded to bf16, fp32 sums; measured 2.3e-3 .. 3.4e-3)."""
import numpy as np
import pytest
import torch

import paper_2511_00413_amd as T
import workloads as W
from oracle import meta as M
from oracle import ssm as S
from tt_testutil import rel_l2

pytestmark = pytest.mark.gpu


def _inputs(n, hk, hv, seed):
    g_ = torch.Generator().manual_seed(seed)
    q = torch.randn((n, hk, 128), generator=g_)
    k = torch.randn((n, hk, 128), generator=g_)
    q = (q / q.norm(dim=-1, keepdim=True)).to(torch.bfloat16)
    k = (k / k.norm(dim=-1, keepdim=True)).to(torch.bfloat16)
    v = torch.randn((n, hv, 128), generator=g_).to(torch.bfloat16)
    g = -(torch.rand((n, hv), generator=g_) * 0.2 + 0.005)
    beta = torch.rand((n, hv), generator=g_) * 0.8 + 0.1
    d_o = torch.randn((n, hv, 128), generator=g_).to(torch.bfloat16)
    return q, k, v, g, beta, d_o


def _check(tree, hk, hv, seed):
    m = M.dfs_meta(tree.parent, tree.seg_len)
    n = m["n_tokens"]
    q, k, v, g, beta, d_o = _inputs(n, hk, hv, seed)
    plan = T.tree_gdn_plan(tree.parent, tree.seg_len)
    print(f"[case] gdn bwd n={n} hk={hk} hv={hv}: {plan.n_chunks} chunks, {plan.n_slots} saved states", flush=True)
    got = T.tree_gdn_bwd(q.cuda(), k.cuda(), v.cuda(), g.cuda(), beta.cuda(), d_o.cuda(), plan)
    torch.cuda.synchronize()
    got = [t.float().cpu().numpy() for t in got]
    want = S.gdn_tree_bwd(q.float().numpy(), k.float().numpy(), v.float().numpy(), g.numpy(), beta.numpy(), m["tok_pred"],
                          d_o.float().numpy())
    for name, a, b, tol in zip(("dq", "dk", "dv", "dg", "dbeta"), got, want, (8e-3, 8e-3, 8e-3, 8e-3, 8e-3)):
        e = rel_l2(a, b)
        print(f"   {name}: rel-L2 {e:.2e}", flush=True)
        assert np.isfinite(a).all(), name
        assert e <= tol, (name, e)


@pytest.mark.parametrize("seed", range(3))
def test_level_schedule_against_sequence_order(seed):
    """The backward with the level schedule (forward walk and reverse walk one launch each over all levels, sibling
    subtrees side by side; state gradients of a slot's readers stored per segment and added in list order) against
    the walk over all chunks in sequence order.  dv and the per-chunk work are identical; where several readers'
    gradients meet, the two walks add them in a different association, so the comparison is to fp32 rounding of the
    sums (1e-5 relative on fp32 outputs, equal up to one bf16 ulp on a few bf16 elements), not bit for bit.  Also
    checks run-to-run reproducibility of the scheduled walk and the gradient of the initial state."""
    t = W.random_tree(940 + seed, n_nodes=9 + 7 * seed, lo=1, hi=150, n_roots=1 + seed % 2, p_zero=0.15)
    m = M.dfs_meta(t.parent, t.seg_len)
    n = m["n_tokens"]
    q, k, v, g, beta, d_o = (x.cuda() for x in _inputs(n, 2, 4, 30 + seed))
    plan = T.tree_gdn_plan(t.parent, t.seg_len).to_device()
    init = torch.randn((4, 128, 128), generator=torch.Generator().manual_seed(seed)).cuda() * 0.1
    print(f"[case] gdn bwd schedule n={n}: {plan.n_chunks} chunks in {plan.n_segments} segments, {plan.n_levels} levels", flush=True)
    plan.parallel = True
    par = T.tree_gdn_bwd(q, k, v, g, beta, d_o, plan, initial_state=init, want_d_initial_state=True)
    par2 = T.tree_gdn_bwd(q, k, v, g, beta, d_o, plan, initial_state=init, want_d_initial_state=True)
    plan.parallel = False
    seq = T.tree_gdn_bwd(q, k, v, g, beta, d_o, plan, initial_state=init, want_d_initial_state=True)
    torch.cuda.synchronize()
    for name, a, b, c in zip(("dq", "dk", "dv", "dg", "dbeta", "d_initial_state"), par, par2, seq):
        assert torch.equal(a, b), f"{name}: the scheduled walk is not reproducible"
        e = rel_l2(a.float().cpu().numpy(), c.float().cpu().numpy())
        print(f"   {name}: scheduled vs sequence order rel-L2 {e:.2e}", flush=True)
        assert e <= (2e-3 if a.dtype == torch.bfloat16 else 1e-4), (name, e)


@pytest.mark.parametrize("parallel", [True, False])
def test_passes_of_key_head_groups(parallel):
    """A workspace too small for all heads makes the call run in passes of whole key-head groups (here 3 key heads x 2
    value heads: one, two or all three key heads per pass).  The heads are independent, so every output must be
    bit-identical whatever the pass size -- with the state gateway in both directions, with and without the level
    schedule; below the smallest size the call is refused."""
    t = W.random_tree(977, n_nodes=12, lo=1, hi=140, n_roots=2, p_zero=0.1)
    m = M.dfs_meta(t.parent, t.seg_len)
    n, hk, hv = m["n_tokens"], 3, 6
    q, k, v, g, beta, d_o = (x.cuda() for x in _inputs(n, hk, hv, 41))
    cap = [i for i in range(len(t.seg_len)) if t.seg_len[i] > 0][:2]
    plan = T.tree_gdn_plan(t.parent, t.seg_len, capture_nodes=cap).to_device()
    plan.parallel = parallel
    gen = torch.Generator().manual_seed(5)
    init = (torch.randn((hv, 128, 128), generator=gen) * 0.1).cuda()
    d_state = (torch.randn((plan.n_capture, hv, 128, 128), generator=gen) * 0.1).cuda()
    full = T.tree_gdn_bwd_workspace(n, hk, hv, plan)
    least = T.tree_gdn_bwd_workspace(n, hk, hv, plan, smallest=True)
    assert least < full
    print(f"[case] gdn bwd passes n={n} hk={hk} hv={hv} schedule={parallel}: workspace {least} .. {full} bytes", flush=True)

    def run(nbytes):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        out = T.tree_gdn_bwd(q, k, v, g, beta, d_o, plan, initial_state=init, d_state_out=d_state, want_d_initial_state=True,
                             workspace=ws)
        torch.cuda.synchronize()
        return out

    ref = run(full)
    for nbytes in (least, (least + full) // 2 + 4096, full - 16):
        got = run(nbytes)
        for name, a, b in zip(("dq", "dk", "dv", "dg", "dbeta", "d_initial_state"), got, ref):
            assert torch.equal(a, b), (name, nbytes)
    with pytest.raises(T.TreeTrainError) as e:
        run(least - 256)
    assert e.value.status == -6


def test_chain_partial_chunks():
    """One sequence of 150 tokens: chunks of 64, 64, 22; then a 1-token sequence."""
    _check(W._mk([-1], [150], [1], "chain"), 1, 2, 0)
    _check(W._mk([-1], [1], [1], "one"), 1, 1, 1)


@pytest.mark.parametrize("seed", range(4))
def test_random_trees(seed):
    t = W.random_tree(880 + seed, n_nodes=6 + 4 * seed, lo=1, hi=150, n_roots=1 + seed % 2, p_zero=0.15)
    _check(t, 2, 4, seed)


def test_branch_point_inside_deep_tree():
    """Several children per node and zero-length nodes: slots are reused, gradients meet at branch points."""
    t = W.random_tree(991, n_nodes=24, lo=0, hi=90, n_roots=2, p_zero=0.2)
    _check(t, 1, 2, 7)


@pytest.mark.parametrize("hk,hv", [(3, 3), (2, 8), (8, 8)])
def test_head_layouts(hk, hv):
    """One value head per key head (no group sum), four per key head, and a head count that is a multiple of
    eight (the workgroup-to-head mapping differs there)."""
    t = W.random_tree(870 + hv, n_nodes=7, lo=1, hi=100, p_zero=0.1)
    _check(t, hk, hv, 40 + hk)


def test_chunk_boundary_lengths():
    """Node lengths at and around the chunk size (63, 64, 65, 128, 129), a zero-length node between two others,
    two roots: chunks of full and of one-token length, branch points at chunk ends."""
    parent = [-1, 0, 0, 1, 1, 2, -1, 6, 7]
    seg = [64, 63, 65, 128, 1, 0, 129, 0, 2]
    _check(W._mk(parent, seg, [1] * len(seg), "boundaries"), 1, 2, 77)


@pytest.mark.parametrize("n_nodes,hk,hv", [(3, 42, 84), (4, 32, 64), (11, 32, 64), (12, 32, 64), (16, 32, 96), (1, 127, 381), (3, 171, 171)])
def test_value_heads_of_a_workgroup(n_nodes, hk, hv):
    """From 128 (chunk, key head) pairs on, one workgroup takes all value heads of a key head and sums dq and dk on chip;
    below, every value head has a workgroup of its own.  Both sides of that line, two and three value heads per key head
    and one; passes over a part of the key heads give the same bits."""
    parent = [-1] + [(i - 1) // 2 for i in range(1, n_nodes)]
    tree = W._mk(parent, [1 + (5 * i) % 9 for i in range(n_nodes)], [1] * n_nodes, "short nodes")
    _check(tree, hk, hv, 55)
    plan = T.tree_gdn_plan(tree.parent, tree.seg_len).to_device()
    assert plan.n_chunks == n_nodes
    n = sum(tree.seg_len)
    ins = [x.cuda() for x in _inputs(n, hk, hv, 56)]
    outs = []
    for smallest in (False, True):
        ws = torch.empty(T.tree_gdn_bwd_workspace(n, hk, hv, plan, smallest=smallest), dtype=torch.uint8, device="cuda")
        outs.append(T.tree_gdn_bwd(*ins, plan, workspace=ws))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*outs))


@pytest.mark.parametrize("rep", [3, 4])
def test_value_heads_of_a_workgroup_full_chunks(rep):
    """The same form with full chunks and chunks of 1, 36 and 63 tokens, three and four value heads per key head: some key
    heads against the oracle; with a state that enters and one that is handed on, against those heads alone (a call of so
    few pairs takes one value head per workgroup), and over passes of one key head bit for bit."""
    parent, seg = [-1, 0, 0, 2, 2, 4], [63, 64, 65, 129, 1, 100]
    hk, hv, n = 40, 40 * rep, sum(seg)
    q, k, v, g, beta, d_o = _inputs(n, hk, hv, 60 + rep)
    heads = [0, 17, 39]
    vheads = [h * rep + r for h in heads for r in range(rep)]
    plan = T.tree_gdn_plan(parent, seg).to_device()
    assert plan.n_chunks * hk >= 128 and plan.n_chunks * len(heads) < 128
    print(f"[case] gdn bwd n={n} hk={hk} hv={hv}: {plan.n_chunks} chunks", flush=True)
    part = lambda got: [x.float().cpu().numpy()[:, heads if i < 2 else vheads] for i, x in enumerate(got)]      # noqa: E731
    got = part(T.tree_gdn_bwd(*(x.cuda() for x in (q, k, v, g, beta, d_o)), plan))
    sub = [x[:, heads] for x in (q, k)] + [x[:, vheads] for x in (v, g, beta, d_o)]
    want = S.gdn_tree_bwd(*(x.float().numpy() for x in sub[:5]), M.dfs_meta(parent, seg)["tok_pred"], sub[5].float().numpy())
    for name, a, b in zip(("dq", "dk", "dv", "dg", "dbeta"), got, want):
        assert rel_l2(a, b) <= 8e-3, (name, rel_l2(a, b))
    # with the gateway in both directions
    plan = T.tree_gdn_plan(parent, seg, capture_nodes=[3]).to_device()
    gen = torch.Generator().manual_seed(rep)
    init = torch.randn((hv, 128, 128), generator=gen) * 0.1
    d_state = torch.randn((1, hv, 128, 128), generator=gen) * 0.1

    def run(ins, init, d_state, smallest=False):
        hk, hv = ins[0].shape[1], ins[2].shape[1]
        ws = torch.empty(T.tree_gdn_bwd_workspace(n, hk, hv, plan, smallest=smallest), dtype=torch.uint8, device="cuda")
        return T.tree_gdn_bwd(*(x.contiguous().cuda() for x in ins), plan, initial_state=init.cuda(), d_state_out=d_state.contiguous().cuda(),
                              want_d_initial_state=True, workspace=ws)

    whole = run((q, k, v, g, beta, d_o), init, d_state)
    passes = run((q, k, v, g, beta, d_o), init, d_state, smallest=True)
    alone = run(sub, init[vheads], d_state[:, vheads])
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(whole, passes))
    for i, (a, b) in enumerate(zip(whole, alone)):
        a = a[vheads] if i == 5 else a[:, heads if i < 2 else vheads]
        # the same products; dq and dk summed over the value heads before or after they leave the chip, then rounded to bf16 once
        e = rel_l2(a.float().cpu().numpy(), b.float().cpu().numpy())
        assert e <= (2e-3 if a.dtype == torch.bfloat16 else 1e-5), (i, e)


def _spine(n):
    """A spine of n branch points: every node has a leaf and the next spine node as children."""
    parent, seg, at = [-1], [3], 0
    for i in range(n):
        parent += [at, at]
        seg += [1 + i % 3, 2 + (i % 5) * 31]
        at = len(parent) - 1
    return W._mk(parent, seg, [1] * len(seg), "spine")


def test_more_levels_than_a_launch_lists():
    """40 dependency levels: segments wait for their parents' states and for their readers' gradients inside one launch;
    the reverse walk orders up to 32 levels longest segment first."""
    t = _spine(40)
    assert T.tree_gdn_plan(t.parent, t.seg_len).n_levels > 32
    _check(t, 1, 2, 13)


def test_two_streams_at_once():
    """Two calls in flight on two streams, each with its own workspace and flags: the results of each alone, bit for bit."""
    trees = [_spine(12), W.random_tree(996, n_nodes=30, lo=1, hi=200, n_roots=2)]
    ins, plans, alone = [], [], []
    for i, t in enumerate(trees):
        n = sum(t.seg_len)
        ins.append([x.cuda() for x in _inputs(n, 8, 16, 90 + i)])
        plans.append(T.tree_gdn_plan(t.parent, t.seg_len).to_device())
        alone.append(T.tree_gdn_bwd(*ins[i], plans[i]))
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in trees]
    for _ in range(3):
        outs = [None, None]
        for i, st in enumerate(streams):
            with torch.cuda.stream(st):
                outs[i] = T.tree_gdn_bwd(*ins[i], plans[i])
        torch.cuda.synchronize()
        for got, want in zip(outs, alone):
            assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("hk,hv", [(1, 2), (2, 4), (3, 12), (10, 20)])
def test_two_streams_at_once_rows_of_any_length(hk, hv):
    """Rows of the walks' grids that are no multiple of eight workgroups: a segment and the one it waits for then run on different
    XCDs.  Forward and backward of two trees in flight on two streams: the results of each alone, bit for bit."""
    trees = [_spine(12), W.random_tree(996, n_nodes=30, lo=1, hi=200, n_roots=2)]
    ins, plans, alone = [], [], []

    def both(i):
        return (T.tree_gdn_fwd(*ins[i][:5], plans[i]),) + T.tree_gdn_bwd(*ins[i], plans[i])

    for i, t in enumerate(trees):
        ins.append([x.cuda() for x in _inputs(sum(t.seg_len), hk, hv, 190 + i)])
        plans.append(T.tree_gdn_plan(t.parent, t.seg_len).to_device())
        alone.append(both(i))
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in trees]
    for _ in range(3):
        outs = [None, None]
        for i, st in enumerate(streams):
            with torch.cuda.stream(st):
                outs[i] = both(i)
        torch.cuda.synchronize()
        for got, want in zip(outs, alone):
            assert all(torch.equal(a, b) for a, b in zip(got, want))


def test_a_wait_that_gives_up_leaves_nan():
    """A chunk program that does not fit its schedule: a state that no segment saves, a gradient that no reader stores.  The walks'
    bounded waits end, what depends on them is NaN and the rest is as it should be."""
    seg = [70, 30, 40]
    ins = [x.cuda() for x in _inputs(sum(seg), 1, 2, 5)]
    plan = T.tree_gdn_plan([-1, 0, 0], seg).to_device()
    o, (dq, dk, dv, dg, db) = T.tree_gdn_fwd(*ins[:5], plan), T.tree_gdn_bwd(*ins, plan)
    torch.cuda.synchronize()
    saved = plan.device["chunk_dst"].clone()
    plan.device["chunk_dst"].fill_(-1)                # the root's segment saves nothing: its children wait in vain
    print("[case] gdn: nobody saves the children's state", flush=True)
    o2, (dq2, dk2, dv2, dg2, db2) = T.tree_gdn_fwd(*ins[:5], plan), T.tree_gdn_bwd(*ins, plan)
    torch.cuda.synchronize()
    assert torch.equal(o2[:70], o[:70]) and torch.equal(dq2[:70], dq[:70])
    assert all(x[70:].isnan().all() for x in (o2, dq2, dg2, db2))
    plan.device["chunk_dst"].copy_(saved)
    plan.device["chunk_src"].clamp_(max=-1)           # the children start from zero and store no gradient: the root waits in vain
    print("[case] gdn: nobody stores the root's gradient", flush=True)
    dq3, dk3, dv3, dg3, db3 = T.tree_gdn_bwd(*ins, plan)
    torch.cuda.synchronize()
    assert all(x[70:].isfinite().all() for x in (dq3, dk3, dv3, dg3, db3))
    assert torch.equal(dq3[:70], dq[:70]) and all(x[:70].isnan().all() for x in (dk3, dv3, dg3, db3))


def test_walks_of_two_and_of_four_waves():
    """Levels of up to 128 walks (segments x heads) run with two waves per workgroup and two that copy for them, wider ones with four:
    levels of 2 segments of 64 and of 65 heads, a node of more chunks than a wave holds scalars of, chunks of 1, 7, 40 and 64 tokens.
    A head's arithmetic is the same in both, so its results are, bit for bit, those of that head alone; which are the oracle's."""
    parent, seg = [-1, 0, 0, 1, 1], [65 * 64 + 7, 40, 70, 1, 129]
    tree = W._mk(parent, seg, [1] * 5, "long")
    _check(tree, 1, 1, 21)
    plan = T.tree_gdn_plan(parent, seg, capture_nodes=[1]).to_device()
    gen = torch.Generator().manual_seed(8)
    ins = list(_inputs(sum(seg), 65, 65, 22)) + [torch.randn((65, 128, 128), generator=gen) * 0.1, torch.randn((1, 65, 128, 128), generator=gen) * 0.1]

    def run(lo, hi):
        x = [t[lo:hi] if i == 6 else t[:, lo:hi] for i, t in enumerate(ins)]
        x = [t.contiguous().cuda() for t in x]
        return T.tree_gdn_bwd(*x[:6], plan, initial_state=x[6], d_state_out=x[7], want_d_initial_state=True)

    wide, narrow = run(0, 65), {h: run(h, h + 1) for h in (0, 37, 64)}
    both = run(0, 64)
    torch.cuda.synchronize()
    for h, alone in narrow.items():
        for i, (a, b, c) in enumerate(zip(wide, both, alone)):
            cut = (lambda t, h=h, i=i: t[h:h + 1] if i == 5 else t[:, h:h + 1])
            assert torch.equal(cut(a), c), (h, i)
            assert h == 64 or torch.equal(cut(b), c), (h, i)


def test_more_segments_than_a_launch_has_rows():
    """70 roots, 65500 branches of the first and what is below one of them: 65572 segments in three levels, walked by two launches whose
    places go on where the first one's ended.  Against the walk over all chunks in sequence order: the same bits, but for the gradients of
    the first root's three tokens.  There 65500 readers' gradients are added in another order: sqrt(65500) 2^-24 = 1.5e-5 of the
    sum, by which one in 250 of its entries is rounded to the other bf16 neighbour (2^-8) on its way into the products: 2.5e-4 in them,
    1e-3 behind another rounding to bf16.  Bounds: four times that."""
    parent = [-1] * 70 + [0] * 65500 + [70, 70, 71]
    seg = [3] * 70 + [1] * 65500 + [2, 66, 5]
    plan = T.tree_gdn_plan(parent, seg).to_device()
    assert plan.n_segments > 65535 and plan.n_levels == 3
    ins = [x.cuda() for x in _inputs(sum(seg), 1, 1, 17)]
    print(f"[case] gdn {plan.n_segments} segments", flush=True)
    got = (T.tree_gdn_fwd(*ins[:5], plan),) + T.tree_gdn_bwd(*ins, plan)
    torch.cuda.synchronize()
    plan.parallel = False
    print("[case] gdn in sequence", flush=True)
    want = (T.tree_gdn_fwd(*ins[:5], plan),) + T.tree_gdn_bwd(*ins, plan)
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0])
    for a, b in zip(got[1:], want[1:]):
        assert torch.equal(a[3:], b[3:])
        assert rel_l2(a[:3].float().cpu().numpy(), b[:3].float().cpu().numpy()) <= (4e-3 if a.dtype == torch.bfloat16 else 1e-3)
