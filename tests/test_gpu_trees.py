"""The forward of small forests filed tree after tree (trees.hip) against the C oracle, at the sizes where its row groups,
unit tiles, weight slabs and waves have remainders, and at the limits of what it takes."""
import numpy as np
import pytest

from workloads import make_forest, make_values, chain_forest, star_forest, perfect_kary_tree, relabel
from gpu_util import run_gpu_forward

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


def _lay_out(trees):
    off = np.concatenate([[0], np.cumsum([t.shape[0] for t in trees])])
    return np.concatenate([np.where(t < 0, -1, t + o) for t, o in zip(trees, off)]).astype(np.int32)


def _word_order(p, seed):
    """Ids inside every tree in any order."""
    cuts = np.append(np.flatnonzero(p < 0), p.shape[0])
    return _lay_out([relabel(np.where(p[a:b] < 0, -1, p[a:b] - a).astype(np.int32), seed + int(a))[0]
                     for a, b in zip(cuts[:-1], cuts[1:])])


def _broom(k):
    """A root with k children that have one leaf each: k rows on the middle level."""
    return np.concatenate([[-1], np.zeros(k), 1 + np.arange(k)]).astype(np.int32)


def _spine(k):
    """k levels: a path whose every node has a leaf beside the next one."""
    p, at = [-1], 0
    for _ in range(k - 1):
        p += [at, at]
        at = len(p) - 1
    return np.array(p, dtype=np.int32)


def _forward_whole(p, x, W, U, b, dtype, save=False):
    """(h, c, gates, fgate, inputs as the GPU sees them) of a forward that has to run as whole trees, into buffers of NaN."""
    import torch
    import paper_1904_07421_amd as J
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    n, H = p.shape[0], U.shape[1]
    dev = [torch.from_numpy(v).cuda().to(dt) for v in (x, W, U)] + [torch.from_numpy(b).cuda()]
    seen = [v.float().cpu().numpy() for v in dev[:3]] + [b]
    out = [torch.full((n, w), float("nan"), dtype=t, device="cuda") for w, t in ((H, dt), (H, torch.float32), (3 * H, dt), (H, dt))]
    s = J.jitdb_schedule(torch.from_numpy(p).cuda())
    J.jitdb_profile_start(4096)
    try:
        if save:
            J.jitdb_treelstm_forward_train(*dev, s, out=tuple(out))
        else:
            J.jitdb_treelstm_forward(*dev, s, out=tuple(out[:2]))
        torch.cuda.synchronize()
    finally:
        prof = J.jitdb_profile_stop()
    assert prof["trees"]["launches"] == 1 and prof["thin_internal"]["launches"] == prof["internal"]["launches"] == 0
    return [v.float().cpu().numpy() for v in out] + [seen]


def _check_whole(c_oracle, p, D, H, dtype, save=False):
    """States of every node against the oracle and, with `save`, the gates of the first and the last trees (about 1000 and 800
    nodes); the bounds are the forward's, but for the gates of nodes with many children."""
    x, W, U, b = make_values(1, p.shape[0], "random", D=D, H=H)
    h, c, gates, fgate, seen = _forward_whole(p, x, W, U, b, dtype, save)
    ho, co, _ = c_oracle(p, *seen)
    assert np.abs(h - ho).max() <= TOL[dtype]
    assert np.abs(c - co).max() <= TOL[dtype] * max(1.0, np.abs(co).max() / (8.0 if dtype == "bf16" else 50.0))
    if not save:
        return
    from oracle import treelstm_backward_oracle as B
    n, has = p.shape[0], p >= 0
    assert np.isfinite(gates).all() and np.isfinite(fgate[has]).all()
    assert np.isnan(fgate[~has]).all()                                # rows of roots stay as handed in
    upto = np.maximum.accumulate(np.maximum(p, np.arange(n)))
    np.maximum.at(upto, p[has], np.flatnonzero(has))                  # the farthest id that an id so far is tied to
    cuts = np.append(1 + np.flatnonzero(np.maximum.accumulate(upto) == np.arange(n)), 0)
    first, last = cuts[cuts >= min(n, 1000)].min(), cuts[cuts <= max(0, n - 800)].max()
    for lo, hi in ((0, first), (max(first, last), n)):
        if lo == hi:
            continue
        part = np.where(p[lo:hi] < 0, -1, p[lo:hi] - lo).astype(np.int32)
        hp, _, go, fo = B.forward_saved(part, seen[0][lo:hi], *seen[1:])
        bound = np.full_like(go, TOL[dtype])
        if dtype == "bf16":
            # A sum of children's h is an operand of 8 bits, off by up to 2^-9 of itself: of 120 children it is past 20, and with its
            # rounding alone (rounded by hand, in fp64) the gates of such a node are 0.016 to 0.032 off.
            hs, up = np.zeros_like(hp), part >= 0
            np.add.at(hs, part[up], hp[up])
            bound += 2.0 ** -9 * (np.abs(hs) @ np.abs(seen[2][:3 * H]).T) * np.repeat([0.25, 0.25, 1.0], H)    # slopes of the gates
        assert (np.abs(gates[lo:hi] - go) <= bound).all()
        assert np.abs(fgate[lo:hi] - fo)[part >= 0].max() <= TOL[dtype]


FORESTS = {
    "one-tree": lambda: perfect_kary_tree(2, 4),
    "leaves-and-stars": lambda: _lay_out([np.full(1, -1, np.int32)] * 3 + [star_forest(k) for k in (2, 5, 6, 17, 18, 34, 70)]),
    # 4, 5, 16, 17, 32, 33 rows of one level inside a block, levels of all sizes above
    "row-groups": lambda: _lay_out([perfect_kary_tree(2, 5)] + [_broom(k) for k in (4, 5, 16, 17, 32, 33, 65)] * 2),
    "word-order": lambda: _word_order(make_forest(2), 3),
    # 32 levels, two trees wide; sequences of up to 12 nodes leave chain levels on top
    "deep": lambda: _lay_out([chain_forest(31), star_forest(4)] * 5 + [_lay_out([perfect_kary_tree(2, 2)])]),
    "many": lambda: _lay_out([make_forest(1)] * 700),
    # 24 levels and few nodes a block: h and f c stay in LDS; every remainder of a group of 16 and of 32 rows
    "near": lambda: _lay_out([perfect_kary_tree(2, 5)] + [_broom(k) for k in (4, 5, 16, 17, 32, 33)] * 2 + [_spine(24)]),
    # ... with trees of up to 97 nodes, which leave little of LDS for f's weights
    "near-full": lambda: _lay_out([_spine(24)] + [_broom(k) for k in (4, 5, 17, 20, 33, 48)]),
    # a tree of 241 nodes: through memory, fp32 from H of 65 on, bf16 from 128; every remainder of a group of 64 rows
    "far": lambda: _lay_out([_spine(31)] + [_broom(k) for k in (4, 5, 15, 16, 17, 36, 64, 65, 68, 120)]),
    # ... in blocks that own many nodes besides: through memory from H of 17 (fp32) and 50 (bf16) on
    "far-many": lambda: _lay_out([make_forest(1)] * 600 + [_broom(k) for k in (4, 5, 15, 16, 17, 36, 64, 65, 68, 120)] + [_spine(24)]),
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("forest,D,H", [
    ("one-tree", 300, 150), ("leaves-and-stars", 7, 33), ("row-groups", 128, 16), ("row-groups", 129, 99), ("word-order", 300, 150),
    ("word-order", 225, 256), ("deep", 44, 50), ("many", 320, 128), ("row-groups", 300, 240), ("word-order", 31, 256),
])
def test_trees_in_one_block_each(c_oracle, forest, D, H, dtype):
    import torch
    import paper_1904_07421_amd as J
    p = FORESTS[forest]()
    x, W, U, b = make_values(1, p.shape[0], "random", D=D, H=H)
    J.jitdb_profile_start(256)
    try:
        s, h, c, seen = run_gpu_forward(p, x, W, U, b, dtype)
    finally:
        prof = J.jitdb_profile_stop()
    launches = {k: v["launches"] for k, v in prof.items() if isinstance(v, dict)}
    print(f"trees {forest} D={D} H={H} {dtype} N={p.shape[0]} L={s.n_levels} launches={launches}", flush=True)
    assert launches["trees"] == 1 and launches["thin_internal"] == launches["internal"] == 0
    ho, co, _ = c_oracle(p, *seen)
    eh, ec = np.abs(h - ho).max(), np.abs(c - co).max()
    # |c| grows with the arity: the flat bound holds up to max|c| = 8 (bf16) / 50 (fp32), in proportion beyond
    assert eh <= TOL[dtype] and ec <= TOL[dtype] * max(1.0, np.abs(co).max() / (8.0 if dtype == "bf16" else 50.0))
    torch.cuda.synchronize()


@pytest.mark.parametrize("save", [False, True])
@pytest.mark.parametrize("dtype,D", [("f32", D) for D in (64, 65, 112, 113, 160, 161, 200, 256, 257, 320)] +
                         [("bf16", D) for D in (128, 129, 224, 225, 320, 321, 393, 512, 513, 600, 640)])
def test_every_width_of_the_x_part(c_oracle, dtype, D, save):
    """Each instance of the x part at both ends of its widths, leaves and inner nodes, with and without saved gates."""
    p, H = FORESTS["word-order"](), 100
    print(f"x part {dtype} D={D} save={save} N={p.shape[0]}", flush=True)
    _check_whole(c_oracle, p, D, H, dtype, save)


@pytest.mark.parametrize("D,H", [(3, 150), (7, 64), (8, 65), (9, 150), (127, 130), (129, 80), (203, 150), (223, 200), (224, 200)])
def test_x_part_over_several_groups(c_oracle, D, H):
    """bf16 rows through LDS: blocks that take several groups of 32 rows (one unit tile to fetch for in the last block of some
    H), last pieces of every length, D below one piece."""
    p = _lay_out([make_forest(1)] * 350)
    print(f"x part D={D} H={H} N={p.shape[0]}", flush=True)
    _check_whole(c_oracle, p, D, H, "bf16")


@pytest.mark.parametrize("trees,D,H,save", [(350, 130, 150, False), (350, 160, 99, True), (350, 192, 200, True), (350, 222, 65, False), (2440, 130, 16, True),
                                            (2440, 222, 16, False)])
def test_x_part_of_even_widths_past_128(c_oracle, trees, D, H, save):
    """bf16 rows of more than 128 and at most 224 columns, an even number: in operand layout, from 160 000 nodes on through LDS (odd
    ones and rows of whole lines always)."""
    p = _lay_out([make_forest(1)] * trees)
    print(f"x part D={D} H={H} N={p.shape[0]} save={save}", flush=True)
    assert (p.shape[0] >= 160000) == (trees > 2000)
    _check_whole(c_oracle, p, D, H, "bf16", save)


RECURRENT = [("near", "f32", (16, 17, 64, 65, 127, 128, 129, 160, 161)),
             ("near", "bf16", (16, 50, 64, 65, 128, 129, 160, 161, 192, 193, 208, 209, 240, 256)),
             ("near-full", "f32", (129, 160)), ("near-full", "bf16", (161, 192)),
             ("far", "f32", (65, 127, 128, 129, 161, 256)), ("far", "bf16", (128, 129, 160, 161, 192, 193, 208, 209, 240, 256)),
             ("far-many", "f32", (17, 64)), ("far-many", "bf16", (50, 64, 65))]


@pytest.mark.parametrize("save", [False, True])
@pytest.mark.parametrize("forest,dtype,H", [(f, t, H) for f, t, widths in RECURRENT for H in widths])
def test_every_width_of_the_recurrent_part(c_oracle, dtype, H, forest, save):
    """Each instance that keeps the recurrent weights in registers at both ends of its widths, child sums through LDS ("near") and
    through memory ("far", and bf16 from 193 units on), all and some of f's weights in LDS; in fp32 past those widths, and from 129
    units on where rows do not fit LDS, the kernel that reads them from L2."""
    p, D = FORESTS[forest](), 24
    print(f"recurrent part {dtype} H={H} {forest} save={save} N={p.shape[0]}", flush=True)
    _check_whole(c_oracle, p, D, H, dtype, save)


@pytest.mark.parametrize("what", ["wide-x", "wide-h", "long-tree", "scrambled"])
def test_what_does_not_fit_runs_level_by_level(c_oracle, what):
    """D past the largest instance, a tree longer than one block should take, ids all over the forest."""
    import paper_1904_07421_amd as J
    p = _lay_out([perfect_kary_tree(2, 8), make_forest(1)]) if what == "long-tree" else make_forest(2)
    if what == "scrambled":
        p = relabel(p, 9)[0]
    x, W, U, b = make_values(1, p.shape[0], "random", D=700 if what == "wide-x" else 40, H=260 if what == "wide-h" else 40)
    J.jitdb_profile_start(4096)
    try:
        s, h, c, seen = run_gpu_forward(p, x, W, U, b, "f32")
    finally:
        prof = J.jitdb_profile_stop()
    ho, co, _ = c_oracle(p, *seen)
    assert prof["trees"]["launches"] == 0
    assert np.abs(h - ho).max() <= 1e-4 and np.abs(c - co).max() <= 1e-4 * max(1.0, np.abs(co).max() / 50.0)


@pytest.mark.parametrize("appended", [False, True])
def test_a_typed_table_as_a_plain_schedule(c_oracle, appended):
    """One cell on a table filed by (height, signature): any order inside a level is a valid batch, and a tree's nodes of a
    level are no longer neighbours."""
    import torch
    import paper_1904_07421_amd as J
    p = FORESTS["word-order"]()
    sig = (np.arange(p.shape[0]) % 3).astype(np.int32)
    s = J.jitdb_schedule_typed(torch.from_numpy(p).cuda(), torch.from_numpy(sig).cuda(), 3)
    if appended:
        more = perfect_kary_tree(2, 3)
        s, p = J.jitdb_schedule_append(s, torch.from_numpy(more).cuda()), _lay_out([p, more])
    x, W, U, b = make_values(1, p.shape[0], "random", D=40, H=48)
    print(f"typed table as a plain schedule N={p.shape[0]} appended={appended}", flush=True)
    h, c = J.jitdb_treelstm_forward(*(torch.from_numpy(v).cuda() for v in (x, W, U, b)), s)
    ho, co, _ = c_oracle(p, x, W, U, b)
    assert np.abs(h.cpu().numpy() - ho).max() <= 1e-4
    assert np.abs(c.cpu().numpy() - co).max() <= 1e-4 * max(1.0, np.abs(co).max() / 50.0)


@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_infinite_weights_saturate_gates(dtype):
    """An infinite weight on one unit's gates: that gate is 0 or 1 (u: -1 or 1), not NaN, in every node (D of one weight slab)."""
    import torch
    import paper_1904_07421_amd as J
    p, D, H = FORESTS["row-groups"](), 8, 33
    x, W, U, b = (torch.from_numpy(v).cuda().to(getattr(torch, dtype)) for v in make_values(1, p.shape[0], "random", D=D, H=H))
    x[:, 0] = 1.0                                         # (0 times the weight is NaN by right)
    for g, v in enumerate((float("-inf"), float("inf"), float("-inf"), float("inf"))):
        W[g * H + 5, 0] = v                               # i = 0, o = 1, u = -1, f = 1: c = 0, h = 0
    h, c = J.jitdb_treelstm_forward(x, W, U, b.float(), J.jitdb_schedule(torch.from_numpy(p).cuda()))
    print(f"infinite weights {dtype} N={p.shape[0]}", flush=True)
    assert bool(torch.isfinite(h).all()) and bool(torch.isfinite(c).all())
    assert bool((h[:, 5] == 0).all()) and bool((c[:, 5] == 0).all())


def _forward_of(s, p, D=40, H=48):
    """(h, c, inputs, launches of the one-block form) of a forward on s."""
    import torch
    import paper_1904_07421_amd as J
    x, W, U, b = make_values(1, p.shape[0], "random", D=D, H=H)
    J.jitdb_profile_start(4096)
    try:
        h, c = J.jitdb_treelstm_forward(*(torch.from_numpy(v).cuda() for v in (x, W, U, b)), s)
        torch.cuda.synchronize()
    finally:
        prof = J.jitdb_profile_stop()
    return h.cpu().numpy(), c.cpu().numpy(), (x, W, U, b), prof["trees"]["launches"]


@pytest.mark.parametrize("how", ["by-hand", "stale", "kept"])
def test_a_tree_window_counts_with_its_tag_only(c_oracle, how):
    """A schedule without a window is not one with whatever its struct holds there; one that is kept takes both along."""
    import torch
    import paper_1904_07421_amd as J
    p = FORESTS["word-order"]()
    filed = J.jitdb_schedule(torch.from_numpy(p).cuda())
    assert 0 < filed.struct.tree_window <= 256
    if how == "kept":
        s = J.Schedule(p.shape[0], "cuda")
        for k in ("height", "level_ptr", "perm", "inv_perm", "child_ptr", "child_idx"):
            getattr(s, k).copy_(getattr(filed, k))
        s.host_level_ptr[:], s.host_level_kids[:] = filed.host_level_ptr, filed.host_level_kids
        s.n_levels, s.n_edges = filed.n_levels, filed.n_edges
        for k in ("n_levels", "n_edges", "tree_window", "tree_tag"):
            setattr(s.struct, k, getattr(filed.struct, k))
    else:
        p = relabel(p, 9)[0]
        if how == "stale":
            p = np.append(p, np.int32(-1))
        s = J.jitdb_schedule(torch.from_numpy(p).cuda())
        if how == "by-hand":                          # (a scrambled forest small enough for one block is all one run of trees)
            s.struct.tree_window = 40
        else:
            s.struct.tree_window, s.struct.tree_tag = filed.struct.tree_window, filed.struct.tree_tag
    print(f"tree window {how} N={p.shape[0]} window={s.struct.tree_window}", flush=True)
    h, c, seen, launches = _forward_of(s, p)
    ho, co, _ = c_oracle(p, *seen)
    assert launches == (1 if how == "kept" else 0)
    assert np.abs(h - ho).max() <= 1e-4 and np.abs(c - co).max() <= 1e-4 * max(1.0, np.abs(co).max() / 50.0)
    if how != "kept":
        more = torch.from_numpy(perfect_kary_tree(2, 3)).cuda()
        assert J.jitdb_schedule_append(s, more).struct.tree_window == 0


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_workspace_without_room_for_whole_trees(c_oracle, dtype):
    """A table's workspace serves a plain forest of its size, level by level; less than that is refused."""
    import torch
    import paper_1904_07421_amd as J
    p, D, H = FORESTS["word-order"](), 40, 150
    n = p.shape[0]
    x, W, U, b = make_values(1, n, "random", D=D, H=H)
    s, h1, c1, seen = run_gpu_forward(p, x, W, U, b, dtype)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    code = J.JITDB_F32 if dtype == "f32" else J.JITDB_BF16
    sizes = [J.jitdb_treelstm_typed_workspace_bytes(n, s.n_edges, D, H, code, k) for k in (2, 3)]
    least = 2 * sizes[0] - sizes[1]                       # less the second cell's weights
    dev = [torch.from_numpy(v).cuda().to(dt) for v in (x, W, U)] + [torch.from_numpy(b).cuda()]
    assert least < J.jitdb_treelstm_workspace_bytes(n, s.n_edges, D, H, code)
    ho, co, _ = c_oracle(p, *seen)
    for size in (sizes[0], least):
        print(f"workspace without room for whole trees {dtype} N={n} {size}", flush=True)
        ws = torch.empty(size + 4096, dtype=torch.uint8, device="cuda").fill_(0xA5)
        h, c = J.jitdb_treelstm_forward(*dev, s, workspace=ws[:size])
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0xA5).all())
        assert np.abs(h.float().cpu().numpy() - ho).max() <= TOL[dtype]
        assert np.abs(c.cpu().numpy() - co).max() <= TOL[dtype] * max(1.0, np.abs(co).max() / (8.0 if dtype == "bf16" else 50.0))
    with pytest.raises(J.JitdbError) as e:
        J.jitdb_treelstm_forward(*dev, s, workspace=ws[:least - 256])
    assert e.value.code == -5


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("what,H,whole", [
    ("one tree of 250 nodes", 240, False), ("one tree of 250 nodes", 40, True),        # one block for all of it, wide cells
    ("interleaved", 150, False), ("filed", 150, True),                                 # the same trees, ids over each other or not
    ("chains, narrow x", 150, False), ("chains", 150, True),
])
def test_whole_trees_where_they_are_the_faster_form(c_oracle, what, H, whole, dtype):
    """Both forms give the oracle's states; which one runs goes by the estimate of their times."""
    import paper_1904_07421_amd as J
    rng = np.random.default_rng(3)
    small = _lay_out([perfect_kary_tree(2, 3)] * 16)
    p = {"one tree of 250 nodes": lambda: np.array([-1] + [int(rng.integers(v)) for v in range(1, 250)], np.int32),
         "interleaved": lambda: relabel(small, 5)[0], "filed": lambda: small,
         "chains, narrow x": lambda: _lay_out([chain_forest(10 + k % 50) for k in range(4000)]),
         "chains": lambda: _lay_out([chain_forest(10 + k % 50) for k in range(400)])}[what]()
    D = {"chains, narrow x": 16, "chains": 300}.get(what, 100)
    x, W, U, b = make_values(1, p.shape[0], "random", D=D, H=H)
    J.jitdb_profile_start(8192)
    try:
        s, h, c, seen = run_gpu_forward(p, x, W, U, b, dtype)
    finally:
        prof = J.jitdb_profile_stop()
    print(f"form {what} H={H} {dtype} N={p.shape[0]} whole={prof['trees']['launches']}", flush=True)
    assert 0 < s.struct.tree_window <= 256
    assert (prof["trees"]["launches"] == 1) == whole
    ho, co, _ = c_oracle(p, *seen)
    assert np.abs(h - ho).max() <= TOL[dtype]
    assert np.abs(c - co).max() <= TOL[dtype] * max(1.0, np.abs(co).max() / (8.0 if dtype == "bf16" else 50.0))
