"""GPU parity: tree attention forward/backward through the C ABI against the per-branch CPU oracle.

Two assertions per output (tt_testutil.ATTN_TOL): the relative L2 over the whole tensor (fp32 path 1e-5;
bf16 path 1e-2 for O and LSE, 2e-2 for dQ/dK/dV) and the largest per-row error -- per (query token, head)
for O and dQ, per (key token, kv head) for dK and dV, largest absolute difference for LSE -- because the
equivalence the method claims holds per token (Eq. 6) and the gradient sum per key (Eq. 5): one wrong row
must fail.  dQ and dK rows get an absolute budget for what the rounding of the saved O (an input of the backward
call, in the I/O dtype) can contribute (tt_testutil.dq_allowance / dk_allowance).  The oracle consumes the same (bf16-rounded) inputs upcast to fp32."""
import numpy as np
import pytest
import torch

import paper_2511_00413_amd as T
import workloads as W
from oracle import attention as A
from oracle import meta as M
from tt_testutil import assert_attention_close, dk_allowance, dq_allowance

pytestmark = pytest.mark.gpu



def _full_parity(tree, dims, seed, scale=None, reference_kernels=False, label=""):
    from gpu_util import gpu_attention
    meta = T.tree_build_meta(tree.parent, tree.seg_len, tree.trained)
    om = M.dfs_meta(tree.parent, tree.seg_len, tree.trained)
    n = meta.n_tokens
    q, k, v, do = W.attn_inputs(n, n, dims, seed)
    print(f"[case] {label} {tree.name} N={n} hq={dims.hq} hkv={dims.hkv} d={dims.d} {dims.dtype} ref={reference_kernels}", flush=True)
    got = gpu_attention(meta, q, k, v, do, scale=scale, reference_kernels=reference_kernels)
    want = A.branches(om, q.float(), k.float(), v.float(), do.float(), scale=scale)
    sc = dims.d ** -0.5 if scale is None else scale
    dk_allow = dk_allowance(q.float().numpy(), k.float().numpy(), want["lse"], M.mask_chunks(om), do.float().numpy(), want["o"],
                            sc, dims.dtype) if 0 < n <= 8192 else None
    errs, _ = assert_attention_close(got, {key: want[key] for key in ("o", "lse", "dq", "dk", "dv")}, dims.dtype,
                                     dq_allow=_dq_allow(do, want["o"], k, scale, dims), dk_allow=dk_allow)
    return errs


def _dq_allow(do, o_ref, k, scale, dims):
    """dq_allowance for whole tensors: d_o, o_ref [n, hq, d]; k [n_keys, hkv, d] (every key a query may see)."""
    if k.shape[0] == 0:
        return None
    kmax = np.repeat(np.linalg.norm(k.float().numpy(), axis=-1).max(axis=0), dims.hq // dims.hkv)      # [hq]
    return dq_allowance(do.float().numpy(), o_ref, kmax[None, :], dims.d ** -0.5 if scale is None else scale, dims.dtype)


def test_cfg1_fp32_worked_tree():
    _full_parity(W.tree_cfg1(), W.DIMS[1], 1, label="cfg1")


@pytest.mark.parametrize("seed", range(6))
def test_fp32_random_trees(seed):
    t = W.random_tree(50 + seed, n_nodes=2 + 3 * seed, lo=1, hi=90, n_roots=1 + seed % 2, p_zero=0.15)
    if t.n_tokens == 0:
        pytest.skip("empty tree drawn")
    hq, hkv, d = [(4, 4, 64), (8, 2, 128), (6, 3, 72), (2, 1, 256), (4, 2, 8), (8, 8, 32)][seed]
    _full_parity(t, W.AttnDims(hq, hkv, d, "fp32", 1.0), seed, scale=0.2 if seed % 2 else None, label="fp32-random")


@pytest.mark.parametrize("ref", [True, False], ids=["reference-kernels", "mfma"])
@pytest.mark.parametrize("seed", range(4))
def test_bf16_random_trees(seed, ref):
    # several 64/128-token tiles per node, ragged tails, zero-length nodes, forests
    t = W.random_tree(70 + seed, n_nodes=3 + 4 * seed, lo=1, hi=400, n_roots=1 + seed % 2, p_zero=0.1)
    hq, hkv = [(4, 1), (8, 2), (4, 4), (16, 2)][seed]
    _full_parity(t, W.AttnDims(hq, hkv, 128, "bf16", 0.5), seed, reference_kernels=ref, label="bf16-random")


@pytest.mark.parametrize("ref", [True, False], ids=["reference-kernels", "mfma"])
def test_bf16_rows_small_by_cancellation(ref):
    """Trees in which most queries see one to three keys (nodes of 1 .. 3 tokens, several roots), and wider ones with
    many heads: there dQ_i and the dK rows of the first keys of a root are small by cancellation, and what the
    rounding of the saved O contributes dominates their error.  These shapes (found by a randomized sweep over 1600
    trees) are the ones that need the per-row budgets of dQ and dK; both kernel sets show the same errors on them."""
    for seed, nn, hi, roots, pz, hq, hkv, inseed, scale in [(1100096, 9, 3, 3, 0.0, 8, 8, 96, 0.11), (1100437, 24, 3, 3, 0.0, 8, 8, 437, None),
                                                            (1100197, 12, 3, 2, 0.3, 2, 1, 197, None), (1102897, 18, 3, 3, 0.0, 2, 2, 897, None),
                                                            (1102144, 19, 70, 3, 0.0, 8, 8, 144, None), (1100200, 19, 300, 3, 0.3, 32, 8, 200, None)]:
        t = W.random_tree(seed, n_nodes=nn, lo=1, hi=hi, n_roots=roots, p_zero=pz)
        _full_parity(t, W.AttnDims(hq, hkv, 128, "bf16", 0.5), inseed, scale=scale, reference_kernels=ref, label="cancellation")


def test_bf16_chain_is_causal_attention():
    _full_parity(W.chain_tree([300, 1, 211]), W.AttnDims(4, 2, 128, "bf16", 0.5), 3, label="chain")


def test_bf16_forest_of_chains():
    _full_parity(W.forest_of_chains([130, 64, 1, 257]), W.AttnDims(4, 2, 128, "bf16", 0.5), 4, label="forest")


def test_bf16_single_token_and_tiny():
    _full_parity(W.chain_tree([1]), W.AttnDims(2, 1, 128, "bf16", 0.5), 5, label="one-token")
    _full_parity(W.tree_cfg1(), W.AttnDims(4, 4, 128, "bf16", 0.5), 6, label="cfg1-shape-bf16")


def test_empty_tree_is_a_no_op():
    from gpu_util import gpu_attention
    meta = T.tree_build_meta([-1], [0])
    dims = W.AttnDims(2, 1, 128, "bf16", 0.5)
    q, k, v, do = W.attn_inputs(0, 0, dims, 1)
    got = gpu_attention(meta, q, k, v, do)
    assert got["o"].shape == (0, 2, 128) and got["dk"].shape == (0, 1, 128)


def _prefix_case(dtype, seed, P, vis, chunk, hq, hkv, d, ref=False):
    """Chunk behind a cached prefix vs the oracle on the equivalent whole tree: a root node made
    of the visible prefix tokens with the chunk's roots hanging below it."""
    from gpu_util import gpu_attention
    dims = W.AttnDims(hq, hkv, d, dtype, 0.5 if dtype == "bf16" else 1.0)
    nvis = int(vis.sum())
    meta = T.tree_build_meta(chunk.parent, chunk.seg_len, chunk.trained, n_prefix=P, prefix_visible=vis,
                             root_pos_offset=[nvis] * int((chunk.parent < 0).sum()))
    n = meta.n_tokens
    q, k, v, do = W.attn_inputs(n, n, dims, seed)
    _, kp, vp, _ = W.attn_inputs(1, P, dims, seed + 100)
    print(f"[case] prefix P={P} visible={nvis} N={n} {dtype} ref={ref}", flush=True)
    got = gpu_attention(meta, q, k, v, do, k_prefix=kp, v_prefix=vp, reference_kernels=ref)
    # whole tree: node 0 = visible prefix tokens, chunk nodes shifted by one
    parent = np.concatenate([[-1], np.where(chunk.parent < 0, 0, chunk.parent + 1)]).astype(np.int32)
    seg = np.concatenate([[nvis], chunk.seg_len]).astype(np.int32)
    om = M.dfs_meta(parent, seg)
    assert np.array_equal(om["tok_pos"][nvis:], meta.tok_pos)           # depth-based positions agree
    sel = torch.from_numpy(np.nonzero(vis)[0])
    # oracle order of the chunk tokens equals the library's DFS order (same child order)
    qw = torch.cat([torch.zeros(nvis, hq, d), q.float()])
    dow = torch.cat([torch.zeros(nvis, hq, d), do.float()])
    kw = torch.cat([kp.float()[sel], k.float()])
    vw = torch.cat([vp.float()[sel], v.float()])
    want = A.branches(om, qw, kw, vw, dow)
    ref = dict(o=want["o"][nvis:], lse=want["lse"][:, nvis:], dq=want["dq"][nvis:], dk=want["dk"][nvis:],
               dv=want["dv"][nvis:])
    mine = dict(got)
    if nvis:
        # fp32 accumulators of the visible cached keys: same bounds (the products are bf16 all the same)
        ref["dk_prefix"], ref["dv_prefix"] = want["dk"][:nvis], want["dv"][:nvis]
        mine["dk_prefix"], mine["dv_prefix"] = got["dk_prefix"][sel.numpy()], got["dv_prefix"][sel.numpy()]
    # budgets of the dK rows on the whole tree (the prefix's zero query rows have dO = 0 and add nothing)
    dk_all = dk_allowance(qw.numpy(), kw.numpy(), want["lse"], M.mask_chunks(om), dow.numpy(), want["o"], d ** -0.5, dtype)
    assert_attention_close(mine, ref, dtype, dq_allow=_dq_allow(do, ref["o"], kw, None, dims),
                           dk_allow={"dk": dk_all[nvis:], "dk_prefix": dk_all[:nvis]} if nvis else dk_all)
    hidden = np.nonzero(vis == 0)[0]
    assert np.all(got["dk_prefix"][hidden] == 0) and np.all(got["dv_prefix"][hidden] == 0)
    return meta, (q, k, v, do, kp, vp), got


@pytest.mark.parametrize("dtype,ref", [("fp32", False), ("bf16", True), ("bf16", False)])
def test_partition_prefix(dtype, ref):
    s = W.step_cfg5(seed=3, n_chunk=700, n_prefix=900 + 37, lo=60, hi=300, root_visible=250)
    _prefix_case(dtype, 11, s.n_prefix, s.prefix_visible, s.chunk, 4, 2, 128 if dtype == "bf16" else 64, ref)
    allv = np.ones(200, dtype=np.uint8)
    _prefix_case(dtype, 12, 200, allv, W.chain_tree([150]), 2, 1, 128 if dtype == "bf16" else 64, ref)


@pytest.mark.parametrize("ref", [True, False], ids=["reference-kernels", "mfma"])
def test_first_tile_is_not_the_first_visible_one(ref):
    """The forward and dQ kernels request key tile 0 before they know which tiles a query tile sees.  Cases in which
    that guess is wrong: a prefix whose first 150 tokens are hidden (tile 0 and tile 1 invisible to everybody), and a
    forest of four roots (the queries of the later roots do not see the first root's keys)."""
    vis = np.ones(400, dtype=np.uint8)
    vis[:150] = 0
    _prefix_case("bf16", 21, 400, vis, W.random_tree(31, n_nodes=5, lo=20, hi=200), 4, 2, 128, ref)
    t = W.random_tree(33, n_nodes=9, lo=50, hi=300, n_roots=4, shuffle=False)
    _full_parity(t, W.AttnDims(4, 2, 128, "bf16", 0.5), 5, reference_kernels=ref, label="four-roots")


def test_prefix_gradients_accumulate():
    from gpu_util import gpu_attention
    s = W.step_cfg5(seed=4, n_chunk=300, n_prefix=256, lo=50, hi=120, root_visible=100)
    meta, (q, k, v, do, kp, vp), first = _prefix_case("bf16", 13, s.n_prefix, s.prefix_visible, s.chunk, 4, 2, 128)
    acc = (torch.full(kp.shape, 1.5, dtype=torch.float32, device="cuda"),
           torch.full(kp.shape, -2.0, dtype=torch.float32, device="cuda"))
    again = gpu_attention(meta, q, k, v, do, k_prefix=kp, v_prefix=vp, prefix_acc=acc)
    vis = s.prefix_visible.astype(bool)
    assert np.allclose(again["dk_prefix"][vis], first["dk_prefix"][vis] + 1.5, rtol=0, atol=1e-5)
    assert np.all(again["dv_prefix"][~vis] == -2.0)


def test_deterministic_run_to_run():
    from gpu_util import gpu_attention
    t = W.random_tree(91, n_nodes=9, lo=30, hi=300)
    meta = T.tree_build_meta(t.parent, t.seg_len)
    dims = W.AttnDims(8, 2, 128, "bf16", 0.5)
    q, k, v, do = W.attn_inputs(meta.n_tokens, meta.n_tokens, dims, 9)
    a = gpu_attention(meta, q, k, v, do)
    b = gpu_attention(meta, q, k, v, do)
    for key in ("o", "lse", "dq", "dk", "dv"):
        assert np.array_equal(a[key], b[key]), key


def test_token_strides_of_a_fused_qkv_buffer():
    from gpu_util import gpu_attention, dev, f64
    t = W.random_tree(92, n_nodes=5, lo=20, hi=150)
    meta = T.tree_build_meta(t.parent, t.seg_len)
    n = meta.n_tokens
    dims = W.AttnDims(4, 2, 128, "bf16", 0.5)
    q, k, v, do = W.attn_inputs(n, n, dims, 10)
    plain = gpu_attention(meta, q, k, v, do)
    fused = torch.cat([q.reshape(n, -1), k.reshape(n, -1), v.reshape(n, -1)], dim=1).to("cuda")
    qv = fused[:, :4 * 128].view(n, 4, 128)
    kv = fused[:, 4 * 128:6 * 128].view(n, 2, 128)
    vv = fused[:, 6 * 128:].view(n, 2, 128)
    kend, kmin, kmax = dev(meta.kend), dev(meta.ktile_kend_min), dev(meta.ktile_kend_max)
    o, lse = T.tree_attn_fwd(qv, kv, vv, kend, kmin, kmax)
    dq, dk, dv = T.tree_attn_bwd(qv, kv, vv, kend, kmin, kmax, o, dev(do), lse)
    assert np.array_equal(f64(o), plain["o"]) and np.array_equal(f64(dk), plain["dk"]) and np.array_equal(f64(dq), plain["dq"])


# Short trees, which take one group of waves per workgroup: one key tile, two, odd and even numbers of them, a second root whose
# queries see nothing of the first tiles, up to a workgroup for every compute unit and one beyond.
@pytest.mark.parametrize("segs,parent,hq,hkv", [
    ([1], [-1], 2, 1), ([64], [-1], 2, 2), ([65], [-1], 4, 2), ([129], [-1], 4, 1), ([64, 63, 66], [-1, 0, 0], 4, 2),
    ([70, 90, 64], [-1, -1, 1], 8, 2), ([200, 100, 150, 61], [-1, 0, 0, 2], 4, 4), ([400, 300, 324], [-1, 0, 0], 32, 8),
    ([400, 300, 325], [-1, 0, 0], 32, 8)])
def test_bf16_forward_two_wave_groups(segs, parent, hq, hkv):
    t = W._mk(parent, segs, [1] * len(segs), "two-groups")
    _full_parity(t, W.AttnDims(hq, hkv, 128, "bf16", 0.5), sum(segs), label="two wave groups")


# Two groups of waves per workgroup (at most one workgroup per compute unit; forward from 24 key tiles on, dQ from 32): both
# sides of the lines, and roots of 1, 64, 65, 129 and 224 tokens behind a long one, so that workgroups see one tile (the second
# group none), two, three and more, odd and even numbers, whole and cut by the mask.
@pytest.mark.parametrize("segs,parent,hq,hkv", [
    ([1000, 472], [-1, 0], 4, 2), ([1000, 473], [-1, 0], 4, 2), ([1100, 884], [-1, 0], 2, 2), ([1100, 885], [-1, 0], 2, 1),
    ([1800, 1, 64, 65, 129, 70, 90, 64], [-1, -1, -1, -1, -1, -1, 5, 5], 4, 2),
    ([64, 1, 128, 129, 1800, 200, 100], [-1, -1, -1, -1, -1, 4, 4], 8, 8)])
def test_bf16_two_wave_groups_many_tiles(segs, parent, hq, hkv):
    t = W._mk(parent, segs, [1] * len(segs), "two-groups")
    _full_parity(t, W.AttnDims(hq, hkv, 128, "bf16", 0.5), sum(segs), label="two wave groups, many tiles")


def test_bf16_two_wave_groups_prefix_and_strides():
    """Two groups behind a cached prefix whose first tiles are hidden (the tile requested in advance is the wrong one), the
    largest launch that takes them and the smallest that does not, and token strides of a fused buffer."""
    from gpu_util import gpu_attention, dev, f64
    vis = np.ones(2100, dtype=np.uint8)
    vis[:150] = 0
    vis[700:1000] = 0
    _prefix_case("bf16", 23, 2100, vis, W.random_tree(31, n_nodes=5, lo=20, hi=200), 4, 2, 128)
    for n in (2048, 2049):               # 256 workgroups of two heads (and the planner's in dQ) and 260 of four
        _full_parity(W.random_tree(34, n_nodes=1, lo=n, hi=n), W.AttnDims(16, 2, 128, "bf16", 0.5), 6, label="two wave groups, line")
    t = W.chain_tree([900, 1200])
    meta = T.tree_build_meta(t.parent, t.seg_len)
    q, k, v, do = W.attn_inputs(2100, 2100, W.AttnDims(4, 2, 128, "bf16", 0.5), 10)
    plain = gpu_attention(meta, q, k, v, do)
    fused = torch.cat([x.reshape(2100, -1) for x in (q, k, v)], dim=1).to("cuda")
    qv, kv, vv = (x.unflatten(1, (-1, 128)) for x in fused.split([512, 256, 256], dim=1))
    mask = tuple(dev(x) for x in (meta.kend, meta.ktile_kend_min, meta.ktile_kend_max))
    o, lse = T.tree_attn_fwd(qv, kv, vv, *mask)
    dq, dk, dv = T.tree_attn_bwd(qv, kv, vv, *mask, o, dev(do), lse)
    for x, key in ((o, "o"), (dq, "dq"), (dk, "dk"), (dv, "dv")):
        assert np.array_equal(f64(x), plain[key]), key


# How the dK / dV pass cuts its key tiles (steps are 64-query tiles x query heads of a kv head): at most 12 steps, nothing is cut;
# 13 .. 16, in chunks of 8; more chunks of 8 to 16 than compute units, hence of 16; chunks of up to 32 and beyond.
@pytest.mark.parametrize("segs,parent,hq,hkv", [
    ([700, 68], [-1, 0], 2, 2), ([700, 69], [-1, 0], 2, 2), ([192], [-1], 4, 1), ([193], [-1], 4, 1), ([30, 20, 50, 60], [-1, 0, 0, 1], 64, 8),
    ([500, 120, 100, 80], [-1, 0, 0, 2], 64, 8), ([900, 300, 100], [-1, 0, 1], 32, 4), ([1500, 600, 400], [-1, 0, 0], 32, 8)])
def test_bf16_key_tiles_cut_into_chunks(segs, parent, hq, hkv):
    t = W._mk(parent, segs, [1] * len(segs), "chunks")
    _full_parity(t, W.AttnDims(hq, hkv, 128, "bf16", 0.5), sum(segs) + hq, label="chunks")


@pytest.mark.parametrize("hq,hkv,d", [(2, 2, 64), (6, 2, 128)])
def test_fp32_matrix_kernels_block_edges(hq, hkv, d):
    """Token counts around the 16-wide blocks and the 128 keys of one round of the waves, nodes that start inside a block,
    and cached keys that end inside one."""
    dims = W.AttnDims(hq, hkv, d, "fp32", 1.0)
    # (a single token has dq = dk = 0 by cancellation, <dO, V> - <dO, O> with O = V: nothing to be relative to)
    for segs in ([2], [15], [16], [17], [128], [129], [40, 1, 3, 88], [500, 13]):
        _full_parity(W.chain_tree(segs), dims, sum(segs), label="fp32-chain")
    _full_parity(W.random_tree(641, n_nodes=24, lo=1, hi=30, n_roots=2, p_zero=0.1), dims, 8, label="fp32-short-nodes")
    vis = np.ones(37, dtype=np.uint8)
    vis[5:20] = 0
    _prefix_case("fp32", 22, 37, vis, W.random_tree(642, n_nodes=6, lo=1, hi=50), hq, hkv, d, False)


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_non_finite_values_reach_only_who_sees_them(d):
    """Infinities and NaN in one branch stay out of the rows of every token that does not see it: finite in exactly the
    places where the row-by-row kernels are."""
    from gpu_util import gpu_attention
    tree = W._mk([-1, 0, 0, 1], [21, 30, 45, 9], [1] * 4, "four nodes")
    meta = T.tree_build_meta(tree.parent, tree.seg_len)
    n = meta.n_tokens
    q, k, v, do = W.attn_inputs(n, n, W.AttnDims(2, 1, d, "fp32", 1.0), 3)
    v[25, 0, 3] = float("inf")
    k[30, 0, 1] = float("nan")
    q[70, 1, 2] = float("nan")
    do[90, 0, 5] = float("inf")
    _same_where_finite(*(gpu_attention(meta, q, k, v, do, reference_kernels=r) for r in (False, True)))


def _same_where_finite(got, ref):
    for key in ("o", "lse", "dq", "dk", "dv"):
        fin = np.isfinite(ref[key])
        assert np.array_equal(np.isfinite(got[key]), fin) and np.array_equal(np.isnan(got[key]), np.isnan(ref[key])), key
        # one wave's sums in another order: 1e-5 of the largest entry
        assert fin.any() and not fin.all() and np.abs(got[key][fin] - ref[key][fin]).max() <= 1e-5 * np.abs(ref[key][fin]).max(), key


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nan_key", [16, 32])
def test_fp32_nan_of_the_only_key_a_wave_sees(d, nan_key):
    """A NaN key that opens a 16-key block: for the query of the same token it is the only key of that block, hence of one
    wave, and its NaN has to survive the join of the waves (LSE, and through it dV of the keys in front); a NaN query makes
    every wave's scores NaN."""
    from gpu_util import gpu_attention
    tree = W._mk([-1, 0], [nan_key + 1, 3], [1, 1], "a chain")
    meta = T.tree_build_meta(tree.parent, tree.seg_len)
    n = meta.n_tokens
    q, k, v, do = W.attn_inputs(n, n, W.AttnDims(2, 2, d, "fp32", 1.0), 4)
    k[nan_key, 0, 1] = float("nan")
    q[5, 1, 2] = float("nan")
    got, ref = (gpu_attention(meta, q, k, v, do, reference_kernels=r) for r in (False, True))
    assert np.isnan(ref["lse"][0, nan_key:]).all() and np.isnan(ref["lse"][1, 5])
    _same_where_finite(got, ref)


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_row_without_a_finite_score(d):
    """The only score of query 0 is -inf, which makes its row and its LSE NaN; the other queries see finite keys too."""
    from gpu_util import gpu_attention
    meta = T.tree_build_meta([-1, 0], [20, 3])
    q, k, v, do = W.attn_inputs(23, 23, W.AttnDims(2, 2, d, "fp32", 1.0), 4)
    q[:, 1, 1] = 0.5
    k[0, 1, 1] = -float("inf")
    got, ref = (gpu_attention(meta, q, k, v, do, reference_kernels=r) for r in (False, True))
    assert np.isnan(ref["lse"][1, 0]) and np.isfinite(ref["lse"][1, 1:]).all()
    _same_where_finite(got, ref)


@pytest.mark.parametrize("dtype,d", [("fp32", 64), ("fp32", 128), ("bf16", 128)])
def test_gradients_in_the_place_of_inputs(dtype, d):
    """dq over o, dk over k and dv over v: every kernel is through with a row before it is overwritten."""
    from gpu_util import dev, f64
    t = W.random_tree(95, n_nodes=12, lo=20, hi=200)
    meta = T.tree_build_meta(t.parent, t.seg_len)
    n = meta.n_tokens
    q, k, v, do = (dev(x) for x in W.attn_inputs(n, n, W.AttnDims(4, 2, d, dtype, 1.0), 12))
    mask = tuple(dev(x) for x in (meta.kend, meta.ktile_kend_min, meta.ktile_kend_max))
    o, lse = T.tree_attn_fwd(q, k, v, *mask)
    want = [f64(x) for x in T.tree_attn_bwd(q, k, v, *mask, o, do, lse)]
    got = [f64(x) for x in T.tree_attn_bwd(q, k, v, *mask, o, do, lse, dq=o, dk=k, dv=v)]
    for a, b in zip(got, want):
        # fp32: other kernels, sums in another order (1e-5 of the largest entry); bf16: the same bits
        assert np.abs(a - b).max() <= (1e-5 * np.abs(b).max() if dtype == "fp32" else 0)


@pytest.mark.parametrize("hq,hkv", [(12, 2), (3, 1), (64, 8), (72, 12)])
@pytest.mark.parametrize("n", [33, 95, 129, 577])
def test_bf16_query_heads_that_share_a_workgroup(hq, hkv, n):
    """1, 2 or 4 query heads of a kv head share a workgroup: 4 where a launch has more blocks of 128 queries than the chip has
    compute units (577 tokens of 64 heads), 2 below that, 1 in the smallest launches (33 tokens) and for odd groups of
    heads; last blocks of 1 .. 65 queries, with and without a prefix."""
    parent, segs = [-1, 0, 0, 1, 1], [n // 3, n // 5, n // 4, 1, 0]
    segs[4] = n - sum(segs)
    t = W._mk(parent, segs, [1] * 5, "packed")
    _full_parity(t, W.AttnDims(hq, hkv, 128, "bf16", 0.5), n + hq, label="packed")
    if n == 577:
        vis = np.ones(70, dtype=np.uint8)
        vis[5:9] = 0
        _prefix_case("bf16", hq, 70, vis, t, hq, hkv, 128)


def test_bf16_two_wave_groups_of_four_heads():
    """Two groups of waves and four query heads per workgroup: more blocks of 128 queries x one head than compute units (288),
    but not of 32 queries x four heads (252), and 44 key tiles, most of them a cached prefix with hidden runs."""
    vis = np.ones(2100, dtype=np.uint8)
    vis[:70] = 0
    vis[900:1300] = 0
    parent, segs = [-1, 0, 0, 2], [200, 141, 250, 50]
    _prefix_case("bf16", 25, 2100, vis, W._mk(parent, segs, [1] * 4, "four heads"), 48, 4, 128)


@pytest.mark.parametrize("hq,hkv,n", [(12, 2, 64), (12, 2, 65), (12, 2, 129), (12, 2, 257), (32, 8, 700), (64, 8, 512), (64, 8, 513), (64, 8, 545),
                                      (64, 8, 576), (64, 8, 577)])
def test_bf16_last_queries_one_head_per_workgroup(hq, hkv, n):
    """Where heads share workgroups the last queries' may take one head each: the last 1 .. 64 in launches of two heads that leave
    compute units over (the whole of 64 tokens among them), the last 1 .. 64 of 128 in those of four, and not from 65 on (577: 5 blocks of 64
    heads are more than the compute units).  A line and a tree, and behind a prefix of 24 key tiles and more with two groups of waves."""
    for parent, segs in (([-1], [n]), ([-1, 0, 0], [n // 3, n // 2, n - n // 3 - n // 2])):
        _full_parity(W._mk(parent, segs, [1] * len(segs), "last alone"), W.AttnDims(hq, hkv, 128, "bf16", 0.5), n + hq, label="last alone")
    if n in (65, 129):
        vis = np.ones(1600, dtype=np.uint8)
        vis[64:200] = 0
        _prefix_case("bf16", hq + n, 1600, vis, W._mk([-1], [n], [1], "last alone"), hq, hkv, 128)
