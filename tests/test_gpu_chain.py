"""Chain levels (forward.hip, chain_kernel): many levels in one launch, each row tile waiting for the tiles that hold its children,
against the C oracle: row tiles full and short, more levels than one launch holds, children in any order, with and
without the x part in Z."""
import numpy as np
import pytest

from workloads import make_forest, make_values, chain_forest, relabel
from gpu_util import run_gpu_forward

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


def _lay_out(trees):
    off = np.concatenate([[0], np.cumsum([t.shape[0] for t in trees])])
    return np.concatenate([np.where(t < 0, -1, t + o) for t, o in zip(trees, off)]).astype(np.int32)


FORESTS = {
    "one-chain": lambda: chain_forest(40),
    "tile": lambda: chain_forest(20, 32),
    "tile-and-one": lambda: chain_forest(20, 33),
    "launches": lambda: chain_forest(600, 3),                    # three launches of up to 256 levels
    "ragged": lambda: _lay_out([make_forest(1)] * 5 + [chain_forest(2 + 7 * i % 90) for i in range(300)]),
    # (word 0, 1, 2 .. of the chains side by side in any order: a tile's children lie in many tiles)
    "any-order": lambda: relabel(chain_forest(30, 700), 3)[0],
    "wide": lambda: chain_forest(5, 8192),                       # the most rows a chain level may have
}


@pytest.mark.parametrize("dtype,D,H", [("f32", 20, 50), ("bf16", 20, 50), ("f32", 300, 256), ("bf16", 64, 256),
                                       ("f32", 36, 300), ("bf16", 36, 300), ("bf16", 8, 512)])
@pytest.mark.parametrize("name", list(FORESTS))
def test_chain_levels_in_one_launch(c_oracle, name, dtype, D, H):
    p = FORESTS[name]()
    if p.shape[0] * H > 4_000_000:
        H = max(4, 4_000_000 // p.shape[0])                      # (the oracle's time)
    x, W, U, b = make_values(1, p.shape[0], "random", D=D, H=H)
    print(f"{name} {dtype} N={p.shape[0]} D={D} H={H}", flush=True)
    for _ in range(2):
        s, h, c, seen = run_gpu_forward(p, x, W, U, b, dtype)
        ho, co, _ = c_oracle(p, *seen)
        assert np.abs(h - ho).max() <= TOL[dtype]
        assert np.abs(c - co).max() <= TOL[dtype] * max(1.0, np.abs(co).max() / (8.0 if dtype == "bf16" else 50.0))


def _by_hand(name, s):
    """`s` without what jitdb_schedule says of whole trees, and with positions that are not known or not right."""
    s.struct.tree_window = 0
    n = s.inv_perm.shape[0]
    if name == "none":
        s.struct.inv_perm = None
    elif name == "zeros":
        s.inv_perm.zero_()
    elif name == "far":
        s.inv_perm.fill_(2 ** 31 - 1)
    elif name == "reversed":
        s.inv_perm.copy_(n - 1 - s.inv_perm)
    elif name == "neighbour":                                    # the row tile beside the child's, in the same level
        s.inv_perm.copy_((s.inv_perm + 16) % n)


@pytest.mark.parametrize("dtype,D,H", [("f32", 20, 50), ("bf16", 64, 256), ("f32", 300, 256)])
@pytest.mark.parametrize("name", ["right", "none", "zeros", "far", "reversed", "neighbour"])
def test_positions_that_are_not_the_inverse_of_perm(c_oracle, name, dtype, D, H):
    import torch
    import paper_1904_07421_amd as J
    from gpu_util import bf16_tensor, dev_parent
    p = relabel(chain_forest(30, 700), 3)[0]
    x, W, U, b = make_values(1, p.shape[0], "random", D=D, H=H)
    print(f"by hand: {name} {dtype} N={p.shape[0]} D={D} H={H}", flush=True)
    if dtype == "bf16":
        (xt, xo), (Wt, Wo), (Ut, Uo) = (bf16_tensor(v) for v in (x, W, U))
    else:
        (xt, xo), (Wt, Wo), (Ut, Uo) = ((torch.from_numpy(v).cuda(), v) for v in (x, W, U))
    s = J.jitdb_schedule(dev_parent(p))
    _by_hand(name, s)
    ho, co, _ = c_oracle(p, xo, Wo, Uo, b)
    for _ in range(2):
        h, c = J.jitdb_treelstm_forward(xt, Wt, Ut, torch.from_numpy(b).cuda(), s)
        assert np.abs(h.float().cpu().numpy() - ho).max() <= TOL[dtype] and np.abs(c.cpu().numpy() - co).max() <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_child_two_levels_below(c_oracle, dtype):
    """Levels made by hand that are no heights: half of the chains pass every third level by, so that a node's child may lie two
    levels below it; every node above level 0 has one child."""
    import torch
    import paper_1904_07421_amd as J
    from gpu_util import bf16_tensor, dev_parent
    D, H = 36, 72
    p = _lay_out([chain_forest(20 if i % 2 else 30) for i in range(300)])
    s = J.jitdb_schedule(dev_parent(p))
    hgt = s.height.cpu().numpy()
    tree = np.cumsum(p < 0) - 1                                  # (a tree's ids begin with its root)
    level = np.where(tree % 2 == 1, hgt + hgt // 2, hgt).astype(np.int32)
    assert (np.bincount(level) > 0).all()
    perm = np.lexsort((np.arange(p.size), level)).astype(np.int32)
    inv = np.empty_like(perm)
    inv[perm] = np.arange(p.size, dtype=np.int32)
    rows = np.bincount(level)
    L = rows.size
    s.struct.tree_window = 0
    s.n_levels = s.struct.n_levels = L
    s.height.copy_(torch.from_numpy(level))
    s.perm.copy_(torch.from_numpy(perm))
    s.inv_perm.copy_(torch.from_numpy(inv))
    s.host_level_ptr[:L + 1] = np.concatenate([[0], np.cumsum(rows)])
    s.level_ptr[:L + 1] = torch.from_numpy(s.host_level_ptr[:L + 1]).cuda()
    s.host_level_kids[:L] = np.where(np.arange(L) > 0, rows, 0)
    x, W, U, b = make_values(1, p.shape[0], "random", D=D, H=H)
    print(f"two levels below: {dtype} N={p.shape[0]} L={L}", flush=True)
    if dtype == "bf16":
        (xt, xo), (Wt, Wo), (Ut, Uo) = (bf16_tensor(v) for v in (x, W, U))
    else:
        (xt, xo), (Wt, Wo), (Ut, Uo) = ((torch.from_numpy(v).cuda(), v) for v in (x, W, U))
    ho, co, _ = c_oracle(p, xo, Wo, Uo, b)
    for _ in range(2):
        h, c = J.jitdb_treelstm_forward(xt, Wt, Ut, torch.from_numpy(b).cuda(), s)
        assert np.abs(h.float().cpu().numpy() - ho).max() <= TOL[dtype] and np.abs(c.cpu().numpy() - co).max() <= TOL[dtype]


@pytest.mark.parametrize("whole_trees", [True, False])
@pytest.mark.parametrize("dtype,D,H,wide", [
    ("f32", 20, 256, 3073),          # 1152 bytes of K: alone in tiles of 32 rows
    ("f32", 36, 320, 2449),          # wider than whole trees of fp32 go
    ("f32", 300, 320, 2449),         # 2560 bytes: alone in tiles of 16
    ("bf16", 64, 256, 3100),         # few tiles a level on average: shared ones of 16 rows, alone 32
    ("bf16", 512, 512, 1537),        # 2048 bytes: 32 rows leave room for one block on a CU
])
def test_wide_and_narrow_levels_in_one_forward(c_oracle, dtype, D, H, wide, whole_trees):
    """Levels that go alone, then many that share launches; every level in a launch of its own (event pairs on) takes the same
    tiles and gives the same bits."""
    import torch
    import paper_1904_07421_amd as J
    from gpu_util import bf16_tensor, dev_parent
    p = _lay_out([chain_forest(2 + (i < 100) + (i < 70) * (i % 50) + 270 * (i == 3)) for i in range(wide)])
    x, W, U, b = make_values(1, p.shape[0], "random", D=D, H=H)
    print(f"wide and narrow: {dtype} N={p.shape[0]} D={D} H={H}", flush=True)
    if dtype == "bf16":
        (xt, xo), (Wt, Wo), (Ut, Uo) = (bf16_tensor(v) for v in (x, W, U))
    else:
        (xt, xo), (Wt, Wo), (Ut, Uo) = ((torch.from_numpy(v).cuda(), v) for v in (x, W, U))
    bt = torch.from_numpy(b).cuda()
    s = J.jitdb_schedule(dev_parent(p))
    if not whole_trees:
        s.struct.tree_window = 0
    outs = [J.jitdb_treelstm_forward(xt, Wt, Ut, bt, s) for _ in range(2)]
    outs.append(J.jitdb_treelstm_forward_packed(xt, J.jitdb_treelstm_pack(Wt, Ut, bt), s))
    J.jitdb_profile_start(4096)
    try:
        outs.append(J.jitdb_treelstm_forward(xt, Wt, Ut, bt, s))
        torch.cuda.synchronize()
    finally:
        prof = J.jitdb_profile_stop()
    assert prof["chain"]["launches"] == s.n_levels - 1
    for h, c in outs[1:]:
        assert torch.equal(h, outs[0][0]) and torch.equal(c, outs[0][1])
    ho, co, _ = c_oracle(p, xo, Wo, Uo, b)
    assert np.abs(outs[0][0].float().cpu().numpy() - ho).max() <= TOL[dtype] and np.abs(outs[0][1].cpu().numpy() - co).max() <= TOL[dtype]


@pytest.mark.parametrize("rows", [40, 230])
@pytest.mark.parametrize("dtype,D,H", [("f32", 300, 512), ("f32", 512, 512), ("bf16", 300, 512), ("bf16", 512, 512), ("bf16", 512, 1600)])
def test_rows_of_many_bytes(c_oracle, dtype, D, H, rows):
    """Rows of 1664 to 4224 bytes of K in levels that share a launch; 230 rows a level are enough tiles for bf16 tiles of 32 rows up to
    1840 bytes."""
    p = chain_forest(12, rows)
    x, W, U, b = make_values(1, p.shape[0], "random", D=D, H=H)
    print(f"wide rows: {dtype} N={p.shape[0]} D={D} H={H}", flush=True)
    for _ in range(2):
        s, h, c, seen = run_gpu_forward(p, x, W, U, b, dtype)
        ho, co, _ = c_oracle(p, *seen)
        assert np.abs(h - ho).max() <= TOL[dtype] and np.abs(c - co).max() <= TOL[dtype]
