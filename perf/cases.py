"""The work that users of this library have it do, as cases that can be timed and compared.

A case names one pass through the public entry points (`op`) and the batch it runs on:

  step    jitdb_schedule + jitdb_treelstm_forward for a batch that was not seen before
  packed  a serving loop with fixed weights over batches that return: the schedule comes from a
          ScheduleCache, the forward runs on weights packed beforehand
  append  arriving trees join a schedule that is there already (jitdb_schedule_append)
  typed   several networks in one table: jitdb_schedule_typed + jitdb_treelstm_forward_typed
  nary    binarised trees under an N-ary cell: jitdb_schedule_typed + jitdb_treelstm_forward_cells
  train   one training step: jitdb_schedule + jitdb_treelstm_forward_train + jitdb_treelstm_backward

The forests are synthetic trees of the shapes the library's own configurations use: random recursive
trees ("rrt"), preferential attachment ("pa", the skewed arities of dependency parses), chains, stars and
random trees in turn ("mix"), and trees of bounded arity ("bin", binarised constituency parses).  Node ids
run tree after tree; inside a tree they start at the root, or, with `shuffle`, stand in any order, as word
positions of a parsed sentence do.
"""
import math

import numpy as np
import torch

import paper_1904_07421_amd as J

DTYPES = {"f32": (torch.float32, 4), "bf16": (torch.bfloat16, 2)}


def listed():
    def case(name, op, kind, trees, lo, hi, D, H, dtype, shuffle=False, **more):
        return dict(name=name, op=op, kind=kind, trees=trees, lo=lo, hi=hi, D=D, H=H, dtype=dtype, shuffle=shuffle, **more)
    return [
        # one request of a parser service: a handful of short trees, every buffer allocated by the call
        case("step-tiny-f32", "step", "rrt", 8, 5, 12, 300, 150, "f32", keep=False),
        # the batch size of the paper (256 sentences), fp32
        case("step-sentences-f32", "step", "pa", 256, 4, 32, 300, 150, "f32", keep=True),
        # bulk inference over sentences in bf16, ids in word order
        case("step-batch-bf16", "step", "pa", 4096, 4, 48, 300, 150, "bf16", shuffle=True, keep=True),
        # sequences, flat lists and trees side by side: 128 levels, long child lists
        case("step-mix-f32", "step", "mix", 4096, 8, 128, 300, 256, "f32", keep=True),
        # widths that fit no padding: D not a multiple of 4, H not a multiple of 8
        case("step-odd-bf16", "step", "rrt", 1000, 3, 40, 203, 99, "bf16", keep=True),
        # the largest batch: 2.4 million nodes at H = 512
        case("step-large-bf16", "step", "rrt", 65536, 8, 64, 300, 512, "bf16", keep=True),
        # serving: batches that return, weights that stay
        case("serve-packed-bf16", "packed", "pa", 1024, 4, 48, 300, 256, "bf16", shuffle=True),
        # new requests join a batch that is already scheduled
        case("append-trees", "append", "rrt", 16384, 8, 64, 300, 512, "bf16", new=256),
        # four networks served from one table, one per tree
        case("typed-4-bf16", "typed", "rrt", 8192, 8, 64, 300, 512, "bf16", n_sig=4, per_node=False),
        # binarised constituency trees under one binary cell
        case("nary-2-bf16", "nary", "bin", 8192, 8, 64, 300, 256, "bf16", arity=2),
        # a training step on the paper's batch
        case("train-sentences-f32", "train", "pa", 256, 4, 32, 300, 150, "f32"),
        # a training step on a large batch
        case("train-large-bf16", "train", "rrt", 32768, 8, 64, 300, 512, "bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: tens of nodes to a million, widths 24 to 512 on and off every padding."""
    op = rng.choice(["step", "step", "step", "packed", "append", "typed", "nary", "train", "train"])
    dtype = rng.choice(["f32", "bf16", "bf16"])
    kind = "bin" if op == "nary" else rng.choice(["rrt", "rrt", "pa", "pa", "mix"])
    D = rng.choice([300, 300, _log_int(rng, 24, 512), 4 * _log_int(rng, 6, 128)])
    H = rng.choice([150, 256, 512, _log_int(rng, 24, 512), 8 * _log_int(rng, 3, 64)])
    lo, hi = rng.choice([(1, 12), (4, 32), (4, 48), (8, 64)])
    if kind == "mix":
        lo, hi = 8, rng.choice([32, 64, 128])
    # no dearer than a quarter of the largest forward (bf16) or the same time in fp32
    per_tree = (lo + hi) / 2 * 8.0 * H * (D + H) * (3 if op == "train" else 1)
    most = int((1.4e12 if dtype == "bf16" else 2.5e11) / per_tree)
    trees = _log_int(rng, 8, max(16, min(32768, most)))
    c = dict(op=op, kind=kind, trees=trees, lo=lo, hi=hi, D=D, H=H, dtype=dtype, shuffle=rng.random() < 0.4)
    if op == "step":
        c["keep"] = rng.random() < 0.7
    elif op == "append":
        c["new"] = max(1, _log_int(rng, 1, max(2, trees // 4)))
    elif op == "typed":
        c["n_sig"] = rng.choice([2, 3, 4, 6])
        c["per_node"] = rng.random() < 0.5
    elif op == "nary":
        c["arity"] = rng.choice([2, 2, 3])
    return c


# ---- forests --------------------------------------------------------------------------------
def _grow(kind, sizes, rng, arity):
    """Parents inside each tree, [trees, max size]; column v of a tree holds the parent of its node v."""
    T, n = len(sizes), int(sizes.max())
    par = np.full((T, n), -1, dtype=np.int64)
    v = np.arange(n)
    if kind == "chain":
        par[:] = v - 1
    elif kind == "star":
        par[:, 1:] = 0
    elif kind == "rrt":
        u = rng.random((T, n))
        par[:, 1:] = np.minimum((u[:, 1:] * v[1:]).astype(np.int64), v[1:] - 1)
    elif kind == "pa":                      # p with weight 1 + its children so far: a node, or the end of an edge
        rows = np.arange(T)
        for i in range(1, n):
            r = np.minimum((rng.random(T) * (2 * i - 1)).astype(np.int64), 2 * i - 2)
            par[:, i] = np.where(r < i, r, par[rows, np.maximum(r - i + 1, 0)])
    else:                                   # bin: a uniformly drawn earlier node that still has a free position
        rows = np.arange(T)
        free = np.zeros((T, n + 1), dtype=np.int64)
        n_free = np.ones(T, dtype=np.int64)
        deg = np.zeros((T, n), dtype=np.int64)
        for i in range(1, n):
            at = np.minimum((rng.random(T) * n_free).astype(np.int64), n_free - 1)
            p = free[rows, at]
            par[:, i] = p
            deg[rows, p] += 1
            full = deg[rows, p] == arity
            free[rows, at] = np.where(full, free[rows, n_free - 1], p)
            n_free -= full
            free[rows, n_free] = i
            n_free += 1
    return par


def _forest(case, n_trees, seed):
    """(parent [N] int32 with -1 for roots, tree of every node [N]).  The sizes of the trees belong to the case, their
    shapes to the seed: every seed's batch has the same number of nodes."""
    rng_size, rng = np.random.default_rng(n_trees), np.random.default_rng([seed, n_trees])
    kind, lo, hi = case["kind"], case["lo"], case["hi"]
    kinds = ("chain", "star", "rrt") if kind == "mix" else (kind,)
    parts, parts_size, parts_tree = [], [], []
    for k, name in enumerate(kinds):
        trees = np.arange(k, n_trees, len(kinds))
        if trees.size == 0:
            continue
        sizes = rng_size.integers(lo, (hi if name in ("chain", kind) else min(hi, 64)) + 1, size=trees.size)
        step = max(1, (1 << 22) // int(sizes.max()))                    # bounds the padded table's size
        for at in range(0, trees.size, step):
            s = sizes[at:at + step]
            par = _grow(name, s, rng, case.get("arity", 2))
            parts.append(par[np.arange(par.shape[1])[None, :] < s[:, None]])
        parts_size.append(sizes)
        parts_tree.append(trees)
    local = np.concatenate(parts)
    sizes_g, trees_g = np.concatenate(parts_size), np.concatenate(parts_tree)
    size = np.empty(n_trees, dtype=np.int64)
    size[trees_g] = sizes_g
    start = np.cumsum(size) - size
    base = np.repeat(start[trees_g], sizes_g)                           # first id of the tree, in the parts' order
    where = base + np.arange(local.size) - np.repeat(np.cumsum(sizes_g) - sizes_g, sizes_g)
    parent = np.empty(local.size, dtype=np.int64)
    parent[where] = np.where(local < 0, -1, local + base)
    tree = np.repeat(np.arange(n_trees), size)
    if case["shuffle"]:
        new_of_old = np.empty(parent.size, dtype=np.int64)
        new_of_old[np.argsort(tree + rng.random(parent.size), kind="stable")] = np.arange(parent.size)
        moved = np.empty_like(parent)
        moved[new_of_old] = np.where(parent < 0, -1, new_of_old[np.maximum(parent, 0)])
        parent = moved
    return parent.astype(np.int32), tree


def _signatures(case, parent, tree, seed):
    """One network per tree, or leaves under network 0 and every other node under one of the rest."""
    rng = np.random.default_rng([seed, 7])
    n_sig = case["n_sig"]
    if not case["per_node"]:
        return rng.integers(0, n_sig, size=int(tree[-1]) + 1)[tree].astype(np.int32)
    inner = np.zeros(parent.size, dtype=bool)
    inner[parent[parent >= 0]] = True
    return np.where(inner, rng.integers(1, n_sig, size=parent.size), 0).astype(np.int32)


# ---- what a program has in hand before the call ---------------------------------------------
def _weights(gen, rows, cols, fan_in, dtype):
    k = 1.0 / math.sqrt(fan_in)
    return (torch.rand((rows, cols), generator=gen, device="cuda") * (2 * k) - k).to(dtype)


def prepare(case, seed):
    D, H = case["D"], case["H"]
    dt, _ = DTYPES[case["dtype"]]
    jdt = J.JITDB_F32 if case["dtype"] == "f32" else J.JITDB_BF16
    gen = torch.Generator(device="cuda").manual_seed(seed)
    parent_h, tree = _forest(case, case["trees"], seed)
    n = parent_h.size
    st = {"op": case["op"], "case": case, "parent": torch.from_numpy(parent_h).cuda()}
    if case["op"] == "append":
        new_h, _ = _forest(case, case["new"], seed + 1)
        st["base"] = J.jitdb_schedule(st["parent"])
        st["new"] = torch.from_numpy(new_h).cuda()
        st["out"] = J.Schedule(n + new_h.size, "cuda")
        st["ws"] = torch.empty(J.jitdb_schedule_append_workspace_bytes(n, new_h.size), dtype=torch.uint8, device="cuda")
        return st

    x = torch.randn((n, D), generator=gen, device="cuda", dtype=torch.float32 if n * D < 1 << 28 else dt)
    st["x"] = x.to(dt)
    if case["op"] in ("typed", "nary"):
        n_sig = case.get("n_sig", 1)
        sig = _signatures(case, parent_h, tree, seed) if case["op"] == "typed" else np.zeros(n, dtype=np.int32)
        st["sig"] = torch.from_numpy(sig).cuda()
        st["sched"] = J.jitdb_schedule_typed(st["parent"], st["sig"], n_sig)
        st["ws_s"] = torch.empty(J.jitdb_schedule_typed_workspace_bytes(n, n_sig), dtype=torch.uint8, device="cuda")
    else:
        n_sig = 1
        st["sched"] = J.jitdb_schedule(st["parent"])
        st["ws_s"] = torch.empty(J.jitdb_schedule_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    E = st["sched"].n_edges
    if case["op"] == "nary":
        N = case["arity"]
        st["cells"] = [(J.JITDB_CELL_NARY, N, _weights(gen, (3 + N) * H, D, D, dt), _weights(gen, (3 + N) * H, N * H, N * H, dt),
                        torch.rand((3 + N) * H, generator=gen, device="cuda") - 0.5)]
        need = J.jitdb_treelstm_cells_workspace_bytes(n, E, D, H, jdt, [(J.JITDB_CELL_NARY, N)])
    else:
        W, U = _weights(gen, n_sig * 4 * H, D, D, dt), _weights(gen, n_sig * 4 * H, H, H, dt)
        b = torch.rand(n_sig * 4 * H, generator=gen, device="cuda") - 0.5
        if case["op"] == "typed":
            W, U, b = W.view(n_sig, 4 * H, D), U.view(n_sig, 4 * H, H), b.view(n_sig, 4 * H)
        st["W"], st["U"], st["b"] = W, U, b
        need = J.jitdb_treelstm_typed_workspace_bytes(n, E, D, H, jdt, n_sig)
    if case["op"] == "step" and not case["keep"]:
        return st
    st["ws_f"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    st["hc"] = (torch.empty((n, H), dtype=dt, device="cuda"), torch.empty((n, H), device="cuda"))
    if case["op"] == "packed":
        st["packed"] = J.jitdb_treelstm_pack(W, U, b)
        st["cache"] = J.ScheduleCache(4)
        st["cache"].get(st["parent"])
    elif case["op"] == "train":
        st["hc"] += (torch.empty((n, 3 * H), dtype=dt, device="cuda"), torch.zeros((n, H), dtype=dt, device="cuda"))
        st["gh"] = torch.randn((n, H), generator=gen, device="cuda")
        st["gc"] = torch.randn((n, H), generator=gen, device="cuda")
        st["grads"] = tuple(torch.empty(s, device="cuda") for s in ((n, D), (4 * H, D), (4 * H, H), (4 * H,)))
        st["ws_b"] = torch.empty(J.jitdb_treelstm_backward_workspace_bytes(st["sched"], D, H, jdt), dtype=torch.uint8,
                                 device="cuda")
    return st


def run(st):
    op = st["op"]
    if op == "step":
        if "ws_f" not in st:
            s = J.jitdb_schedule(st["parent"])
            h, c = J.jitdb_treelstm_forward(st["x"], st["W"], st["U"], st["b"], s)
        else:
            s = J.jitdb_schedule(st["parent"], workspace=st["ws_s"], out=st["sched"])
            h, c = J.jitdb_treelstm_forward(st["x"], st["W"], st["U"], st["b"], s, workspace=st["ws_f"], out=st["hc"])
        return {"h": h, "c": c, "perm": s.perm, "height": s.height}
    if op == "packed":
        s, _ = st["cache"].get(st["parent"])
        return J.jitdb_treelstm_forward_packed(st["x"], st["packed"], s, workspace=st["ws_f"], out=st["hc"])
    if op == "append":
        s = J.jitdb_schedule_append(st["base"], st["new"], workspace=st["ws"], out=st["out"])
        return {"height": s.height, "perm": s.perm, "inv_perm": s.inv_perm, "child_ptr": s.child_ptr,
                "child_idx": s.child_idx[:s.n_edges], "n_levels": s.n_levels}
    if op == "typed":
        s = J.jitdb_schedule_typed(st["parent"], st["sig"], st["case"]["n_sig"], workspace=st["ws_s"], out=st["sched"])
        h, c = J.jitdb_treelstm_forward_typed(st["x"], st["W"], st["U"], st["b"], s, workspace=st["ws_f"], out=st["hc"])
        return {"h": h, "c": c, "perm": s.perm, "key": s.key}
    if op == "nary":
        s = J.jitdb_schedule_typed(st["parent"], st["sig"], 1, workspace=st["ws_s"], out=st["sched"])
        return J.jitdb_treelstm_forward_cells(st["x"], st["cells"], s, workspace=st["ws_f"], out=st["hc"])
    s = J.jitdb_schedule(st["parent"], workspace=st["ws_s"], out=st["sched"])
    h, c, gates, fgate = J.jitdb_treelstm_forward_train(st["x"], st["W"], st["U"], st["b"], s, workspace=st["ws_f"],
                                                        out=st["hc"])
    dx, dW, dU, db = J.jitdb_treelstm_backward(st["x"], st["W"], st["U"], s, h, c, gates, fgate, st["gh"], st["gc"],
                                               workspace=st["ws_b"], out=st["grads"])
    return {"h": h, "c": c, "dx": dx, "dW": dW, "dU": dU, "db": db}


def work(case):
    D, H = case["D"], case["H"]
    esz = DTYPES[case["dtype"]][1]
    parent, _ = _forest(case, case["trees"], 0)
    n = parent.size
    if case["op"] == "append":
        m = _forest(case, case["new"], 1)[0].size
        # the base's height, perm, child_ptr, child_idx and the new parents in; six arrays of the joint forest out
        return {"bytes": 4.0 * (4 * n + m + 6 * (n + m)), "flops": 0.0}
    E = int((parent >= 0).sum())
    n_int = int(np.unique(parent[parent >= 0]).size)
    n_leaf = n - n_int
    states = n * H * (esz + 4.0)
    if case["op"] == "nary":
        N = case["arity"]
        weights = (3 + N) * H * ((D + N * H) * esz + 4.0)
        flops = n_leaf * 2.0 * D * 3 * H + n_int * 2.0 * D * (3 + N) * H + E * 2.0 * H * (3 + N) * H
        return {"bytes": 8.0 * n + n * D * esz + weights + states, "flops": flops}
    weights = case.get("n_sig", 1) * 4 * H * ((D + H) * esz + 4.0)
    flops = n_leaf * 2.0 * D * 3 * H + n_int * (2.0 * D * 4 * H + 2.0 * H * 3 * H) + E * 2.0 * H * H
    nbytes = 4.0 * n + n * D * esz + weights + states
    if case["op"] == "typed":
        nbytes += 12.0 * n                       # signatures in, perm and key out
    elif case["op"] == "step":
        nbytes += 8.0 * n                        # perm and height out
    elif case["op"] == "train":                  # cotangents in, gradients out; two products for each of the forward's
        nbytes += 8.0 * n * H + 4.0 * n * D + 4 * H * (D + H + 1) * 4.0
        flops *= 3
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["op"] == "append":
        return "exact"
    # fp32 sums in another order; bf16 operands and stored states (8 bits), fed from level to level
    return {"rel": 1e-5 if case["dtype"] == "f32" else 1e-2}
