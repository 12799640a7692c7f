"""tt_tree_conv_plan (host C++): the successor list of the tree convolution's backward.  Together
with the runs of directly-following tokens it must cover every (token, successor within K-1 steps)
pair of the oracle's predecessor chains exactly once, at the right distance."""
import numpy as np
import pytest

import paper_2511_00413_amd as T
import workloads as W
from oracle import meta as M
from oracle import ssm as S


def _direct_run(tok_pred, first, limit):
    """Tokens first, first+1, ... while each directly follows the one before; at most `limit`."""
    out = [first]
    while len(out) < limit and out[-1] + 1 < len(tok_pred) and tok_pred[out[-1] + 1] == out[-1]:
        out.append(out[-1] + 1)
    return out


def _check(tok_pred, K):
    tok_pred = np.asarray(tok_pred, dtype=np.int32)
    n = len(tok_pred)
    P = S.pred_chain(tok_pred, K)
    want = {(int(P[m][t]), t): m for m in range(1, K) for t in range(n) if P[m][t] >= 0}
    got = {}
    for s in range(n):                                             # what the fast path covers
        for m, t in enumerate(_direct_run(tok_pred, s, K)):
            if m:
                assert (s, t) not in got
                got[(s, t)] = m
    plan = T.tree_conv_plan(tok_pred, K)
    assert np.all(np.diff(plan.fix_tok) > 0) and plan.fix_off[0] == 0 and plan.fix_off[-1] == len(plan.fix_t)
    for f, s in enumerate(plan.fix_tok):
        for e in range(plan.fix_off[f], plan.fix_off[f + 1]):
            t0, r = int(plan.fix_t[e]), int(plan.fix_r[e])
            assert 1 <= r < K
            for m1, t in enumerate(_direct_run(tok_pred, t0, K - r)):
                assert (int(s), t) not in got, "a successor is listed twice"
                got[(int(s), t)] = r + m1
    assert got == want
    return plan


@pytest.mark.parametrize("seed", range(20))
def test_random_trees(seed):
    t = W.random_tree(800 + seed, n_nodes=2 + 2 * seed, lo=1, hi=4, n_roots=1 + seed % 3, p_zero=0.25)
    m = M.dfs_meta(t.parent, t.seg_len)
    for K in (2, 3, 4):
        _check(m["tok_pred"], K)


def test_chain_has_nothing_to_fix_and_star_has():
    m = M.dfs_meta([-1, 0, 1], [3, 4, 5])
    assert len(_check(m["tok_pred"], 4).fix_tok) == 0
    m = M.dfs_meta([-1, 0, 0, 0], [5, 2, 2, 2])                    # tokens 0..4 | 5 6 | 7 8 | 9 10
    plan = _check(m["tok_pred"], 3)
    assert plan.fix_tok.tolist() == [3, 4]                          # the root's last K-1 tokens
    assert plan.fix_t.tolist() == [7, 9, 7, 9] and plan.fix_r.tolist() == [2, 2, 1, 1]


def test_agrees_with_library_meta_and_errors():
    t = W.tree_config(2)
    meta = T.tree_build_meta(t.parent, t.seg_len, t.trained)
    plan = T.tree_conv_plan(meta.tok_pred, 4)
    n_branching_children = int(((meta.tok_pred >= 0) & (meta.tok_pred != np.arange(meta.n_tokens) - 1)).sum())
    assert len(plan.fix_t) == 3 * n_branching_children              # every node here is longer than K-1
    with pytest.raises(T.TreeTrainError) as e:
        T.tree_conv_plan([-1, 0, 1], 5)
    assert e.value.status == -8
    with pytest.raises(T.TreeTrainError) as e:
        T.tree_conv_plan([-1, 2, 0], 3)                              # a predecessor must be an earlier token
    assert e.value.status == -3


def test_backward_workspace_stays_below_its_bound():
    """Tiles are never shorter than the power of two (32 .. 256 tokens) that makes 1024 workgroups of 16-byte lanes: what
    a call of a given shape may need for its partial sums is bounded by that rule, whatever the tile that is used."""
    rng = np.random.default_rng(5)
    for _ in range(2000):
        bf16, k = bool(rng.integers(2)), int(rng.integers(2, 5))
        lane = 8 if bf16 else 4
        c, n = lane * int(10 ** rng.uniform(0, 4)), int(10 ** rng.uniform(0, 6.3))
        tile = 256
        while tile > 32 and -(-n // tile) * (c // lane) < 1024 * 256:
            tile //= 2
        need = T.binding._lib().tt_tree_conv_bwd_workspace(n, c, k, T.binding.DTYPE_BF16 if bf16 else T.binding.DTYPE_FP32)
        assert 0 < need <= -(-n // tile) * (k + 1) * c * 4 + 256, (n, c, k, bf16)
