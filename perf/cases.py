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
