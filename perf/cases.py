"""Performance cases of the tree-training path, through the package's public entry points.

What a training program does with this library, once per layer or once per step and tree: attention forward and
backward over a DFS-serialised tree (bf16; fp32 for numerical verification), attention of a query chunk behind a cached
prefix, attention of a tree cut into partitions, the log-prob loss (scoring, and training with the gradient), rotary
embedding with tree positions, the tree-correct convolution and the gated delta rule.  A case is a dict of plain values;
`n` is the number of tokens (rows) throughout.

Trees are drawn as one of a few shapes whose segment lengths are scaled to exactly `n` tokens, so odd totals and odd
segment lengths are the rule:
  worked    the worked three-leaf tree (root -> A -> {A1, A2}, root -> B), lengths 64:48:32:40:56
  agentic   depth 4, two to four children per node, segment lengths within a factor of eight
  fanout    a shared prefix, sixteen branches, two leaves each (8:2:1)
  chain     a spine of 32 segments with dead-end side chains
"""
import random

import numpy as np
import torch

import paper_2511_00413_amd as T

DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}


# ---- trees ---------------------------------------------------------------------------------------

def _tree(shape, n, tree_seed):
    """(parent, seg_len) of a tree of exactly n tokens."""
    rng = random.Random(tree_seed)
    parent, weight = [], []

    def add(par, w):
        parent.append(par)
        weight.append(w)
        return len(parent) - 1

    if shape == "worked":
        root = add(-1, 64)
        a = add(root, 48)
        add(a, 32)
        add(a, 40)
        add(root, 56)
    elif shape == "agentic":
        def grow(par, level):
            me = add(par, rng.uniform(1.0, 8.0))
            if level < 4:
                for _ in range(rng.randint(2, 4)):
                    grow(me, level + 1)
        grow(-1, 1)
    elif shape == "fanout":
        root = add(-1, 8.0)
        for _ in range(16):
            b = add(root, 2.0)
            add(b, 1.0)
            add(b, 1.0)
    elif shape == "chain":
        prev = -1
        for _ in range(32):
            prev = add(prev, rng.uniform(1.0, 4.0))
            if rng.random() < 0.25:
                side = prev
                for _ in range(rng.randint(1, 3)):
                    side = add(side, rng.uniform(1.0, 4.0))
    else:
        raise ValueError(f"unknown tree shape {shape}")
    edge = np.round(np.cumsum(weight) / sum(weight) * n).astype(np.int64)
    edge[-1] = n
    return np.asarray(parent, np.int32), np.diff(np.concatenate([[0], edge])).astype(np.int32)


def _trained(n_nodes, share, tree_seed):
    rng = random.Random(tree_seed + 1)
    flags = [1 if rng.random() < share else 0 for _ in range(n_nodes)]
    flags[-1] = 1
    return np.asarray(flags, np.uint8)


def _prefix_visible(n_prefix, tree_seed):
    """Half of the cached slice is the trunk (visible); behind it visible and hidden runs alternate."""
    rng = random.Random(tree_seed + 2)
    vis = np.ones(n_prefix, np.uint8)
    pos, flag = n_prefix // 2, 1
    while pos < n_prefix:
        run = rng.randint(max(1, n_prefix // 32), max(2, n_prefix // 8))
        vis[pos:pos + run] = flag
        flag ^= 1
        pos += run
    return vis


def _depth_sum(parent, seg):
    """Sum over tokens of the number of keys a token sees (its depth in tokens, itself included)."""
    start, total = [0] * len(seg), 0
    for i, s in enumerate(int(x) for x in seg):
        start[i] = start[parent[i]] + int(seg[parent[i]]) if parent[i] >= 0 else 0     # parents come first here
        total += s * start[i] + s * (s + 1) // 2
    return total


# ---- cases ---------------------------------------------------------------------------------------

def listed():
    return [
        # fp32 verification of a tiny worked tree (forward + backward): latency and launches
        {"name": "attn_train_fp32_tiny", "kind": "attn_train", "dtype": "fp32", "shape": "worked", "tree_seed": 1, "n": 240,
         "hq": 4, "hkv": 4, "d": 64, "std": 1.0, "fused": False},
        # forward only over one short rollout (scoring a small tree): latency
        {"name": "attn_fwd_small", "kind": "attn_fwd", "dtype": "bf16", "shape": "agentic", "tree_seed": 5, "n": 777,
         "hq": 32, "hkv": 8, "d": 128, "std": 0.5, "fused": False},
        # the ordinary training step: a 16 K-token random tree, forward + backward
        {"name": "attn_train_16k", "kind": "attn_train", "dtype": "bf16", "shape": "agentic", "tree_seed": 117, "n": 16406,
         "hq": 32, "hkv": 8, "d": 128, "std": 0.5, "fused": False},
        # a large agentic fan-out: 8 K shared prefix, 32 leaves, 64 query heads
        {"name": "attn_train_72k", "kind": "attn_train", "dtype": "bf16", "shape": "fanout", "tree_seed": 1, "n": 73728,
         "hq": 64, "hkv": 8, "d": 128, "std": 0.5, "fused": False},
        # the partition step of a tree that does not fit: 32 K-token chunk behind 64 K cached prefix keys, fp32 accumulation
        {"name": "attn_step_32k_64k", "kind": "attn_step", "dtype": "bf16", "shape": "agentic", "tree_seed": 9, "n": 32768,
         "n_prefix": 65536, "hq": 64, "hkv": 8, "d": 128, "std": 0.5},
        # the partition driver on the ordinary tree, cut at about a quarter of its size, forward + backward
        {"name": "attn_partitioned_16k", "kind": "attn_partitioned", "dtype": "bf16", "shape": "agentic", "tree_seed": 117,
         "n": 16406, "capacity": 5120, "hq": 32, "hkv": 8, "d": 128, "std": 0.5},
        # scoring: log-probs of a batch of tokens under an odd vocabulary (rows not on 16-byte boundaries)
        {"name": "loss_fwd_odd_vocab", "kind": "loss_fwd", "dtype": "bf16", "n": 8191, "vocab": 32003, "share": 0.5},
        # training: one 4 K-row chunk of a large vocabulary, loss and gradient together
        {"name": "loss_train_large_vocab", "kind": "loss_train", "dtype": "bf16", "n": 4096, "vocab": 151936, "share": 0.9},
        # rotary embedding of the queries and keys of the ordinary tree
        {"name": "rope_16k", "kind": "rope", "dtype": "bf16", "shape": "agentic", "tree_seed": 117, "n": 16406, "hq": 32,
         "hkv": 8, "d": 128, "inverse": False, "fused": False},
        # convolution in front of a GDN layer, forward + backward
        {"name": "conv_train_16k", "kind": "conv_train", "dtype": "bf16", "shape": "agentic", "tree_seed": 117, "n": 16406,
         "channels": 8192, "taps": 4, "silu": True, "bias": True},
        # gated delta rule of the ordinary tree: forward, and backward
        {"name": "gdn_fwd_16k", "kind": "gdn_fwd", "shape": "agentic", "tree_seed": 117, "n": 16406, "hk": 16, "hv": 32,
         "gateway": False},
        {"name": "gdn_bwd_16k", "kind": "gdn_bwd", "shape": "agentic", "tree_seed": 117, "n": 16406, "hk": 16, "hv": 32,
         "gateway": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["attn_train_fp32", "attn_fwd", "attn_train", "attn_train", "attn_step", "attn_partitioned", "loss_fwd",
                       "loss_train", "rope", "conv_train", "gdn_fwd", "gdn_bwd"])
    shape = rng.choice(["agentic", "agentic", "fanout", "chain"])
    tree_seed = rng.randint(1, 1 << 20)
    hq, hkv = rng.choice([(32, 8), (64, 8), (16, 4), (8, 8)])
    tree = {"shape": shape, "tree_seed": tree_seed}
    if kind == "attn_train_fp32":
        return {"kind": "attn_train", "dtype": "fp32", **tree, "n": _log_int(rng, 128, 2048), "hq": 4, "hkv": rng.choice([2, 4]),
                "d": rng.choice([64, 128]), "std": 1.0, "fused": rng.random() < 0.3}
    if kind in ("attn_fwd", "attn_train"):
        return {"kind": kind, "dtype": "bf16", **tree, "n": _log_int(rng, 256, 65536 if shape != "chain" else 32768), "hq": hq,
                "hkv": hkv, "d": 128, "std": 0.5, "fused": rng.random() < 0.3}
    if kind == "attn_step":
        return {"kind": kind, "dtype": "bf16", **tree, "n": _log_int(rng, 1024, 24576), "n_prefix": _log_int(rng, 1024, 49152),
                "hq": hq, "hkv": hkv, "d": 128, "std": 0.5}
    if kind == "attn_partitioned":
        n = _log_int(rng, 4096, 65536 if shape != "chain" else 32768)
        return {"kind": kind, "dtype": "bf16", **tree, "n": n, "capacity": max(1024, int(n * rng.uniform(0.2, 0.6))), "hq": hq,
                "hkv": hkv, "d": 128, "std": 0.5}
    if kind in ("loss_fwd", "loss_train"):
        vocab = _log_int(rng, 8192, 160000)
        if rng.random() < 0.6:
            vocab = (vocab + 63) // 64 * 64                      # padded vocabularies are the usual ones
        return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "fp32"]), "n": _log_int(rng, 64, 4096), "vocab": vocab,
                "share": rng.choice([0.5, 0.9])}
    if kind == "rope":
        return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "fp32"]), **tree, "n": _log_int(rng, 256, 65536), "hq": hq,
                "hkv": hkv, "d": rng.choice([64, 128, 128]), "inverse": rng.random() < 0.5, "fused": rng.random() < 0.3}
    if kind == "conv_train":
        return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "fp32"]), **tree, "n": _log_int(rng, 256, 32768),
                "channels": rng.choice([1024, 2048, 4096, 6144, 8192]), "taps": rng.choice([4, 4, 3, 2]),
                "silu": rng.random() < 0.8, "bias": rng.random() < 0.7}
    hk, hv = rng.choice([(16, 32), (16, 32), (8, 16), (4, 8), (8, 8)])
    return {"kind": kind, **tree, "n": _log_int(rng, 256, 32768), "hk": hk, "hv": hv, "gateway": rng.random() < 0.3}


# ---- inputs --------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _randn(g, *size, std=1.0, dtype=torch.bfloat16):
    return torch.randn(size, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(dtype)


def _cuda(a):
    return torch.from_numpy(a).to("cuda")


def _qkv(case, g, dtype):
    """q, k, v: tensors of their own, or slices of one fused projection buffer."""
    n, hq, hkv, d, std = case["n"], case["hq"], case["hkv"], case["d"], case.get("std", 0.5)
    if case.get("fused"):
        buf = _randn(g, n, (hq + 2 * hkv) * d, std=std, dtype=dtype)
        q, k, v = buf.split([hq * d, hkv * d, hkv * d], dim=1)
        return q.unflatten(1, (hq, d)), k.unflatten(1, (hkv, d)), v.unflatten(1, (hkv, d))
    return tuple(_randn(g, n, h, d, std=std, dtype=dtype) for h in (hq, hkv, hkv))


def prepare(case, seed):
    g, kind = _gen(seed), case["kind"]
    s = {"kind": kind}
    if kind in ("loss_fwd", "loss_train"):
        n, vocab = case["n"], case["vocab"]
        parent, seg = _tree("agentic", n, vocab)
        meta = T.tree_build_meta(parent, seg, _trained(len(seg), case["share"], vocab))
        s["logits"] = _randn(g, n, vocab, std=2.0, dtype=DTYPES[case["dtype"]])
        s["target"] = torch.randint(0, vocab, (n,), generator=g, device="cuda", dtype=torch.int32)
        s["weight"] = _cuda(meta.tok_weight)
        return s
    parent, seg = _tree(case["shape"], case["n"], case["tree_seed"])
    n = case["n"]
    if kind in ("attn_fwd", "attn_train", "attn_step"):
        n_prefix, vis, off = case.get("n_prefix", 0), None, None
        if n_prefix:
            vis = _prefix_visible(n_prefix, case["tree_seed"])
            off = [int(vis.sum())]
        meta = T.tree_build_meta(parent, seg, root_pos_offset=off, n_prefix=n_prefix, prefix_visible=vis)
        s["mask"] = tuple(_cuda(a) for a in (meta.kend, meta.ktile_kend_min, meta.ktile_kend_max))
        dtype = DTYPES[case["dtype"]]
        s["qkv"] = _qkv(case, g, dtype)
        s["d_o"] = _randn(g, n, case["hq"], case["d"], std=case["std"], dtype=dtype) if kind != "attn_fwd" else None
        s["prefix"] = tuple(_randn(g, n_prefix, case["hkv"], case["d"], std=case["std"], dtype=dtype) for _ in range(2)) if n_prefix else None
    elif kind == "attn_partitioned":
        s["plan"] = T.tree_partition_plan(parent, seg, case["capacity"]).to_device()
        s["qkv"] = _qkv(case, g, torch.bfloat16)
        s["d_o"] = _randn(g, n, case["hq"], case["d"], std=case["std"])
    elif kind == "rope":
        s["q"], s["k"], _ = _qkv(case, g, DTYPES[case["dtype"]])
        s["pos"] = _cuda(T.tree_build_meta(parent, seg).tok_pos)
        s["inverse"] = case["inverse"]
    elif kind == "conv_train":
        c, dtype = case["channels"], DTYPES[case["dtype"]]
        pred = T.tree_build_meta(parent, seg).tok_pred
        s["pred"] = _cuda(pred)
        s["plan"] = T.tree_conv_plan(pred, case["taps"]).to_device()
        s["x"], s["dy"] = _randn(g, n, c, dtype=dtype), _randn(g, n, c, dtype=dtype)
        s["w"] = _randn(g, c, case["taps"], std=0.5, dtype=torch.float32)
        s["b"] = _randn(g, c, std=0.1, dtype=torch.float32) if case["bias"] else None
        s["silu"] = case["silu"]
    else:                                                        # gdn_fwd, gdn_bwd
        hk, hv = case["hk"], case["hv"]
        # with the gateway the tree is one partition: it starts from a parent's state and hands on a leaf's
        cut = [len(seg) - 1] if case["gateway"] else []
        s["plan"] = T.tree_gdn_plan(parent, seg, cut).to_device()
        unit = lambda x: torch.nn.functional.normalize(x, dim=-1).to(torch.bfloat16)      # noqa: E731  (the layer's L2 norm)
        s["q"], s["k"] = (unit(_randn(g, n, hk, 128, dtype=torch.float32)) for _ in range(2))
        s["v"] = _randn(g, n, hv, 128)
        s["g"] = -(0.005 + 0.2 * torch.rand(n, hv, generator=g, device="cuda"))
        s["beta"] = 0.1 + 0.8 * torch.rand(n, hv, generator=g, device="cuda")
        s["d_o"] = _randn(g, n, hv, 128) if kind == "gdn_bwd" else None
        s["state"] = _randn(g, hv, 128, 128, std=0.1, dtype=torch.float32) if case["gateway"] else None
        s["d_state"] = _randn(g, 1, hv, 128, 128, std=0.1, dtype=torch.float32) if case["gateway"] else None
    return s


def run(s):
    kind = s["kind"]
    if kind == "attn_fwd":
        return T.tree_attn_fwd(*s["qkv"], *s["mask"])
    if kind == "attn_train":
        o, lse = T.tree_attn_fwd(*s["qkv"], *s["mask"])
        return (o, lse) + T.tree_attn_bwd(*s["qkv"], *s["mask"], o, s["d_o"], lse)
    if kind == "attn_step":
        kp, vp = s["prefix"]
        dkp, dvp = (torch.zeros(kp.shape, dtype=torch.float32, device=kp.device) for _ in range(2))
        o, lse = T.tree_attn_fwd(*s["qkv"], *s["mask"], k_prefix=kp, v_prefix=vp)
        grads = T.tree_attn_bwd(*s["qkv"], *s["mask"], o, s["d_o"], lse, k_prefix=kp, v_prefix=vp, dk_prefix_acc=dkp, dv_prefix_acc=dvp)
        return (o, lse) + grads + (dkp, dvp)
    if kind == "attn_partitioned":
        o, lse = T.tree_attn_partitioned_fwd(*s["qkv"], s["plan"])
        return (o, lse) + T.tree_attn_partitioned_bwd(*s["qkv"], s["plan"], o, s["d_o"], lse)
    if kind == "loss_fwd":
        return T.tree_weighted_logprob(s["logits"], s["target"], s["weight"])
    if kind == "loss_train":
        return T.tree_weighted_logprob_fwd_bwd(s["logits"], s["target"], s["weight"])
    if kind == "rope":
        return tuple(T.tree_rope(x, s["pos"], inverse=s["inverse"]) for x in (s["q"], s["k"]))
    if kind == "conv_train":
        y = T.tree_conv_fwd(s["x"], s["w"], s["b"], s["pred"], silu=s["silu"])
        return (y,) + T.tree_conv_bwd(s["x"], s["w"], s["b"], s["pred"], s["dy"], s["plan"], silu=s["silu"], want_dbias=s["b"] is not None)
    ins = (s["q"], s["k"], s["v"], s["g"], s["beta"])
    if kind == "gdn_fwd":
        return T.tree_gdn_fwd(*ins, s["plan"], initial_state=s["state"], return_states=s["state"] is not None)
    return T.tree_gdn_bwd(*ins, s["d_o"], s["plan"], initial_state=s["state"], d_state_out=s["d_state"],
                          want_d_initial_state=s["state"] is not None)


# ---- what a pass cannot do without ---------------------------------------------------------------

def work(case):
    kind, n = case["kind"], case["n"]
    e = 2 if case.get("dtype", "bf16") == "bf16" else 4
    if kind.startswith("attn"):
        hq, hkv, d = case["hq"], case["hkv"], case["d"]
        pairs = _depth_sum(*_tree(case["shape"], n, case["tree_seed"]))
        n_prefix = case.get("n_prefix", 0)
        if n_prefix:
            pairs += n * int(_prefix_visible(n_prefix, case["tree_seed"]).sum())
        fwd = n * (2 * hq + 2 * hkv) * d * e + 4 * hq * n + n_prefix * 2 * hkv * d * e
        if kind == "attn_fwd":
            return {"bytes": fwd, "flops": 4.0 * hq * d * pairs}
        # d_o in; dq, dk, dv and the fp32 gradients of the prefix out
        grad = n * (2 * hq + 2 * hkv) * d * e + n_prefix * 2 * hkv * d * 4
        return {"bytes": fwd + grad, "flops": 14.0 * hq * d * pairs}
    if kind == "loss_fwd":
        return {"bytes": n * case["vocab"] * e + 16 * n, "flops": 0}
    if kind == "loss_train":
        return {"bytes": 2 * n * case["vocab"] * e + 16 * n, "flops": 0}
    if kind == "rope":
        return {"bytes": 2 * n * (case["hq"] + case["hkv"]) * case["d"] * e + 4 * n, "flops": 0}
    if kind == "conv_train":
        return {"bytes": 4 * n * case["channels"] * e + 4 * n, "flops": 0}       # x, dy in; y, dx out
    hk, hv = case["hk"], case["hv"]
    gate = hv * 128 * 128 * 4 if case["gateway"] else 0
    # token recurrence: S^T k, rank-1 update, S^T q; its backward redoes the first two and needs two products for each
    if kind == "gdn_fwd":
        return {"bytes": n * (2 * hk + 2 * hv) * 256 + 8 * n * hv + 2 * gate, "flops": 6.0 * 128 * 128 * n * hv}
    return {"bytes": n * (4 * hk + 3 * hv) * 256 + 16 * n * hv + 3 * gate, "flops": 16.0 * 128 * 128 * n * hv}


def tolerance(case):
    """About four times what this path differs by from the same mathematics in fp64 on the same inputs (rel / max measured on
    trees of a few hundred to a few thousand tokens)."""
    kind, bf16 = case["kind"], case.get("dtype", "bf16") == "bf16"
    if kind.startswith("attn"):                 # bf16: one rounding of P, dS and the outputs, 2.4e-3 / 0.1; fp32: 6e-7 / 1.1e-5
        return {"rel": 1e-2, "max": 0.4} if bf16 else {"rel": 3e-6, "max": 5e-5}
    if kind.startswith("gdn"):                  # operands, states and outputs rounded to bf16: 3.5e-3 / 2.5e-2
        return {"rel": 1.4e-2, "max": 0.1}
    if kind == "loss_fwd" or not bf16:          # fp32 results: 1.7e-7 / 1.9e-6 at most (convolution weight gradients)
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 7e-3, "max": 1.6e-2}         # one rounding to bf16: 1.9e-3 / 3.9e-3


# ---- the same results in 64 bits, by plain torch -------------------------------------------------

def _exact_attn(case, s):
    """Node by node: the queries of a node see the tokens of its ancestors (and the visible cached keys) whole and its own
    tokens causally."""
    n, hq, hkv, d = case["n"], case["hq"], case["hkv"], case["d"]
    parent, seg = _tree(case["shape"], n, case["tree_seed"])
    n_prefix = case.get("n_prefix", 0)
    if work(case)["flops"] > 1e14:
        return None
    q, k, v = (x.double().transpose(0, 1) for x in s["qkv"])                   # [heads, tokens, d]
    d_o = None if s["d_o"] is None else s["d_o"].double().transpose(0, 1)
    seen = []
    if n_prefix:
        kp, vp = (x.double().transpose(0, 1) for x in s["prefix"])
        k, v = torch.cat([kp, k], 1), torch.cat([vp, v], 1)
        seen = [_cuda(np.flatnonzero(_prefix_visible(n_prefix, case["tree_seed"])))]
    start = np.concatenate([[0], np.cumsum(seg)])
    o, dq = torch.empty_like(q), torch.zeros_like(q)
    lse = torch.empty(hq, n, dtype=torch.float64, device="cuda")
    dk, dv = torch.zeros_like(k), torch.zeros_like(v)
    scale, g = d ** -0.5, hq // hkv
    for i in range(len(seg)):
        up, a = [], i
        while a >= 0:
            up.append(torch.arange(n_prefix + start[a], n_prefix + start[a + 1], device="cuda"))
            a = int(parent[a])
        keys = torch.cat(seen + up[::-1])
        past = len(keys) - int(seg[i])                                         # keys in front of the node
        step = max(1, (1 << 26) // max(1, len(keys)))
        for h in range(hkv):
            kh, vh, hs = k[h, keys], v[h, keys], slice(h * g, (h + 1) * g)
            dkh, dvh = torch.zeros_like(kh), torch.zeros_like(vh)
            for a in range(int(start[i]), int(start[i + 1]), step):
                b = min(a + step, int(start[i + 1]))
                last = past + torch.arange(a, b, device="cuda") - int(start[i])
                hidden = torch.arange(len(keys), device="cuda")[None, :] > last[:, None]
                for hh in range(hs.start, hs.stop):
                    p = (q[hh, a:b] @ kh.T).mul_(scale).masked_fill_(hidden, -float("inf"))
                    lse[hh, a:b] = p.logsumexp(1)
                    p = p.sub_(lse[hh, a:b, None]).exp_()
                    o[hh, a:b] = p @ vh
                    if d_o is None:
                        continue
                    up_o = d_o[hh, a:b]
                    dvh += p.T @ up_o
                    ds = (up_o @ vh.T).sub_((up_o * o[hh, a:b]).sum(1, keepdim=True)).mul_(p).mul_(scale)
                    dq[hh, a:b] = ds @ kh
                    dkh += ds.T @ q[hh, a:b]
            dk[h].index_add_(0, keys, dkh)
            dv[h].index_add_(0, keys, dvh)
    out = (o.transpose(0, 1), lse)
    if d_o is not None:
        dq, dk, dv = (x.transpose(0, 1) for x in (dq, dk, dv))
        out += (dq, dk[n_prefix:], dv[n_prefix:]) + ((dk[:n_prefix], dv[:n_prefix]) if n_prefix else ())
    return tuple(x.contiguous() for x in out)


def _exact_loss(case, s):
    z, target, w = s["logits"], s["target"].long(), s["weight"].double()
    logp, lse, grad = [], [], []
    for a in range(0, len(z), 512):
        zr, t = z[a:a + 512].double(), target[a:a + 512, None]
        lse.append(zr.logsumexp(1))
        logp.append(zr.gather(1, t)[:, 0] - lse[-1])
        if case["kind"] == "loss_train":
            zr.sub_(lse[-1][:, None]).exp_().scatter_add_(1, t, torch.full(t.shape, -1.0, dtype=zr.dtype, device="cuda"))
            grad.append(zr.mul_(w[a:a + 512, None]))
    logp, lse = torch.cat(logp), torch.cat(lse)
    out = (logp, lse, -(w * logp).sum().reshape(1))
    return out + (torch.cat(grad),) if grad else out


def _exact_rope(s, base=1.0e6):
    out = []
    for x in (s["q"].double(), s["k"].double()):
        half = x.shape[2] // 2
        freq = base ** (-torch.arange(half, dtype=torch.float64, device="cuda") / half)
        ang = (s["pos"].double()[:, None] * freq)[:, None] * (-1.0 if s["inverse"] else 1.0)
        lo, hi, c, sn = x[..., :half], x[..., half:], ang.cos(), ang.sin()
        out.append(torch.cat([lo * c - hi * sn, hi * c + lo * sn], -1))
    return tuple(out)


def _exact_conv(s):
    x, w, dy, pred = s["x"].double(), s["w"].double(), s["dy"].double(), s["pred"].long()
    n, taps = len(x), w.shape[1]
    at, back = [], torch.arange(n, device="cuda")
    for _ in range(taps):                                                      # tokens that have an m-th predecessor, and which
        rows = torch.nonzero(back >= 0)[:, 0]
        at.append((rows, back[rows]))
        back = torch.where(back >= 0, pred[back.clamp(min=0)], back)
    pre = torch.zeros_like(x) if s["b"] is None else s["b"].double().expand_as(x).clone()
    for m, (rows, src) in enumerate(at):
        pre.index_add_(0, rows, x[src] * w[:, taps - 1 - m])
    sig = torch.sigmoid(pre)
    g = dy * sig * (1 + pre * (1 - sig)) if s["silu"] else dy
    dx, dw = torch.zeros_like(x), torch.zeros_like(w)
    for m, (rows, src) in enumerate(at):
        dx.index_add_(0, src, g[rows] * w[:, taps - 1 - m])
        dw[:, taps - 1 - m] = (g[rows] * x[src]).sum(0)
    return pre * sig if s["silu"] else pre, dx, dw, None if s["b"] is None else g.sum(0)


def _exact_gdn(case, s):
    """The token recurrence, and its reverse with the states of one node at a time."""
    n, hk, hv, dim = case["n"], case["hk"], case["hv"], 128
    if n > (24576 if case["kind"] == "gdn_fwd" else 17000):
        return None
    parent, seg = _tree(case["shape"], n, case["tree_seed"])
    start = np.concatenate([[0], np.cumsum(seg)])
    heads = torch.arange(hv, device="cuda") // (hv // hk)
    q, k, v, decay, beta = s["q"].double()[:, heads], s["k"].double()[:, heads], s["v"].double(), s["g"].double().exp(), s["beta"].double()
    scale = dim ** -0.5
    first = torch.zeros(hv, dim, dim, dtype=torch.float64, device="cuda") if s["state"] is None else s["state"].double()

    def walk(i, state):
        states = torch.empty(int(seg[i]) + 1, hv, dim, dim, dtype=torch.float64, device="cuda")
        states[0] = state
        for j in range(int(seg[i])):
            t = int(start[i]) + j
            nxt = torch.mul(states[j], decay[t, :, None, None], out=states[j + 1])
            delta = beta[t, :, None] * (v[t] - torch.bmm(k[t, :, None], nxt)[:, 0])
            nxt.baddbmm_(k[t, :, :, None], delta[:, None])
        return states

    ends, o = [], torch.empty_like(v)
    for i in range(len(seg)):
        states = walk(i, first if parent[i] < 0 else ends[parent[i]])
        a, b = int(start[i]), int(start[i + 1])
        o[a:b] = scale * torch.matmul(q[a:b, :, None], states[1:])[:, :, 0]
        ends.append(states[-1].clone())
    if case["kind"] == "gdn_fwd":
        return o if s["state"] is None else (o, ends[-1][None])
    d_o = s["d_o"].double()
    d_end = [torch.zeros_like(first) for _ in seg]
    if s["d_state"] is not None:
        d_end[-1] += s["d_state"][0].double()
    d_first = torch.zeros_like(first)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    dg, dbeta = torch.empty_like(beta), torch.empty_like(beta)
    for i in reversed(range(len(seg))):
        states, r = walk(i, first if parent[i] < 0 else ends[parent[i]]), d_end[i]
        for j in reversed(range(int(seg[i]))):
            t = int(start[i]) + j
            bt, kt = beta[t, :, None], k[t, :, :, None]
            old = states[j] * decay[t, :, None, None]
            miss = v[t] - torch.bmm(kt.mT, old)[:, 0]
            r = torch.baddbmm(r, scale * q[t, :, :, None], d_o[t, :, None])
            dq[t] = scale * torch.bmm(states[j + 1], d_o[t, :, :, None])[:, :, 0]
            dd = torch.bmm(kt.mT, r)[:, 0]
            dv[t], dbeta[t] = bt * dd, (dd * miss).sum(1)
            dk[t] = torch.bmm(r, (bt * miss)[:, :, None])[:, :, 0] - bt * torch.bmm(old, dd[:, :, None])[:, :, 0]
            r = r - kt * (bt * dd)[:, None]
            dg[t] = (r * old).sum((1, 2))
            r = r * decay[t, :, None, None]
        if parent[i] < 0:
            d_first += r
        else:
            d_end[parent[i]] += r
    dq, dk = (x.unflatten(1, (hk, hv // hk)).sum(2) for x in (dq, dk))
    return (dq, dk, dv, dg, dbeta) + (() if s["state"] is None else (d_first,))


def exact(case, seed):
    """What run returns for these inputs, in float64; None where it would take too long."""
    s, kind = prepare(case, seed), case["kind"]
    if kind.startswith("attn"):
        return _exact_attn(case, s)
    if kind.startswith("loss"):
        return _exact_loss(case, s)
    if kind == "rope":
        return _exact_rope(s)
    return _exact_conv(s) if kind == "conv_train" else _exact_gdn(case, s)
