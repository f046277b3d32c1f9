"""The backward pass at the edges of its tiles and ranges, against the gradient oracle (GPU)."""
import numpy as np
import pytest
import torch

import paper_1904_07421_amd as J
from oracle import treelstm_backward_oracle as B
from workloads import make_values, to_bf16_bits, bf16_bits_to_f32

pytestmark = pytest.mark.gpu

# Relative to the largest entry of each gradient.  fp32: products of a few rounded factors (2^-24 each), sums of at most
# 9000 of them whose errors add up like a random walk: 10 * sqrt(9000) * 2^-24 = 6e-5.  bf16: dz, hs, dhs, ufg, h and the
# gates are rounded (2^-9 each) on a way of at most three levels; five of them in a row and in one direction are 1e-2, twice
# that with the parent's.
TOL = {"f32": 1e-4, "bf16": 2e-2}


def _stars(leaves, kids, chain=0):
    """`leaves` nodes in stars of `kids` leaves (the last one smaller), the stars' centres under a root of `kids`, and so on;
    children before parents; then `chain` lone roots."""
    parent = np.full(leaves, -1, dtype=np.int64)
    level = np.arange(leaves)
    total = leaves
    for _ in range(2):
        groups = -(-len(level) // kids)
        up = total + np.arange(groups)
        parent[level] = up[np.arange(len(level)) // kids]
        parent = np.concatenate([parent, np.full(groups, -1, dtype=np.int64)])
        total += groups
        level = up
    return np.concatenate([parent, np.full(chain, -1, dtype=np.int64)]).astype(np.int32)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("leaves,kids,lone,D,H", [
    (1, 1, 0, 1, 1),             # a chain of three nodes, the narrowest cell
    (64, 3, 0, 127, 64),         # internal rows start on a whole range of 64; [x | 1] fills its 128 columns
    (63, 17, 2, 128, 65),        # ... one short of it, one column more, one gate wider than 64; five chunks of children
    (100, 2, 29, 40, 256),       # the forget gate has column tiles of its own
    (8300, 9, 0, 400, 512),      # enough rows for the 128 x 256 tiles in a level and in dx, too few in the others
])
def test_backward_at_the_edges_of_its_tiles(leaves, kids, lone, D, H, dtype):
    parent = _stars(leaves, kids, lone)
    n = len(parent)
    x, W, U, b = make_values(1, n, "random", D=D, H=H)
    rng = np.random.default_rng(leaves)
    gh = rng.standard_normal((n, H)).astype(np.float32)
    gc = rng.standard_normal((n, H)).astype(np.float32)
    print(f"backward tiles leaves={leaves} kids={kids} D={D} H={H} dtype={dtype} N={n}", flush=True)
    if dtype == "bf16":
        bits = [to_bf16_bits(a) for a in (x, W, U)]
        dev = [torch.from_numpy(t.view(np.int16)).view(torch.bfloat16).cuda() for t in bits]
        seen = [bf16_bits_to_f32(t) for t in bits]
    else:
        dev = [torch.from_numpy(a).cuda() for a in (x, W, U)]
        seen = [x, W, U]
    bd = torch.from_numpy(b).cuda()
    s = J.jitdb_schedule(torch.from_numpy(parent).cuda())
    h, c, gates, fgate = J.jitdb_treelstm_forward_train(*dev, bd, s)
    g = [torch.from_numpy(a).cuda() for a in (gh, gc)]
    got = J.jitdb_treelstm_backward(dev[0], dev[1], dev[2], s, h, c, gates, fgate, *g)
    again = J.jitdb_treelstm_backward(dev[0], dev[1], dev[2], s, h, c, gates, fgate, *g)
    torch.cuda.synchronize()
    want = B.forward_backward(parent, *seen, b, gh, gc)[2:]
    for name, a, a2, r in zip(("dx", "dW", "dU", "db"), got, again, want):
        assert torch.equal(a, a2), name                       # the ranges are added in order
        err = float(np.abs(a.cpu().numpy() - r).max() / max(1.0, np.abs(r).max()))
        print(f"   {name} {err:.2e}", flush=True)
        assert err <= TOL[dtype], (name, err)


def test_partial_sums_stay_inside_the_workspace():
    """Chains: so few leaves that the sums are long ones (cut eight times finer) where those of leaves alone are not."""
    n, D, H = 70000, 64, 1024
    v = torch.arange(n, dtype=torch.int32)
    s = J.jitdb_schedule(torch.where(v % 10 == 0, -1, v - 1).cuda())
    gen = torch.Generator(device="cuda").manual_seed(1)
    rand = lambda *size: torch.randn(size, generator=gen, device="cuda") / size[-1] ** 0.5
    x, W, U, b = rand(n, D).bfloat16(), rand(4 * H, D).bfloat16(), rand(4 * H, H).bfloat16(), rand(4 * H)
    need = J.jitdb_treelstm_backward_workspace_bytes(s, D, H, J.JITDB_BF16)
    buf = torch.full((need + (1 << 29),), 0x5A, dtype=torch.uint8, device="cuda")
    print(f"backward workspace N={n} D={D} H={H} {need >> 20} MiB", flush=True)
    h, c, gates, fgate = J.jitdb_treelstm_forward_train(x, W, U, b, s)
    dx, dW, dU, db = J.jitdb_treelstm_backward(x, W, U, s, h, c, gates, fgate, rand(n, H), None, workspace=buf[:need])
    assert bool((buf[need:] == 0x5A).all())
    assert all(bool(torch.isfinite(g).all()) for g in (dx, dW, dU, db))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("lone,H", [(1, 256), (3, 150), (60, 64), (64, 256)])
def test_an_infinite_cotangent_of_a_leaf_stays_out_of_the_inner_nodes_sums(lone, H, dtype):
    """A lone root is a leaf and nobody's child: its cotangent reaches its own dx row and the i, o, u rows of dW and db, but
    neither dU nor the forget rows.  The last leaf stands right before the inner nodes, wherever that falls in a range."""
    parent, D = _stars(100, 7, lone), 40
    n = len(parent)
    gen = torch.Generator(device="cuda").manual_seed(lone)
    rand = lambda *size: torch.randn(size, generator=gen, device="cuda") / size[-1] ** 0.5
    x, W, U, b = rand(n, D).to(dtype), rand(4 * H, D).to(dtype), rand(4 * H, H).to(dtype), rand(4 * H)
    s = J.jitdb_schedule(torch.from_numpy(parent).cuda())
    h, c, gates, fgate = J.jitdb_treelstm_forward_train(x, W, U, b, s)
    gh = rand(n, H)
    print(f"infinite cotangent N={n} leaves={int(s.host_level_ptr[1])} H={H} {dtype}", flush=True)
    want = J.jitdb_treelstm_backward(x, W, U, s, h, c, gates, fgate, gh, None)
    gh[n - 1, 7] = float("inf")
    dx, dW, dU, db = J.jitdb_treelstm_backward(x, W, U, s, h, c, gates, fgate, gh, None)
    assert not bool(torch.isfinite(dx[n - 1]).all())
    assert torch.equal(dx[:n - 1], want[0][:n - 1])
    assert torch.equal(dU, want[2])
    assert torch.equal(dW[3 * H:], want[1][3 * H:]) and torch.equal(db[3 * H:], want[3][3 * H:])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D,H", [(41, 66), (42, 68), (44, 70), (46, 72), (63, 65)])
def test_rows_that_end_inside_a_piece(D, H, dtype):
    """Rows are read in pieces of 16 bytes; the last one ends after one, two, three or four pairs, or odd."""
    parent = _stars(60, 6)
    n = len(parent)
    x, W, U, b = make_values(1, n, "random", D=D, H=H)
    gh = np.random.default_rng(H).standard_normal((n, H)).astype(np.float32)
    print(f"backward row ends D={D} H={H} dtype={dtype} N={n}", flush=True)
    if dtype == "bf16":
        bits = [to_bf16_bits(a) for a in (x, W, U)]
        dev = [torch.from_numpy(t.view(np.int16)).view(torch.bfloat16).cuda() for t in bits]
        seen = [bf16_bits_to_f32(t) for t in bits]
    else:
        dev = [torch.from_numpy(a).cuda() for a in (x, W, U)]
        seen = [x, W, U]
    s = J.jitdb_schedule(torch.from_numpy(parent).cuda())
    h, c, gates, fgate = J.jitdb_treelstm_forward_train(*dev, torch.from_numpy(b).cuda(), s)
    got = J.jitdb_treelstm_backward(dev[0], dev[1], dev[2], s, h, c, gates, fgate, torch.from_numpy(gh).cuda(), None)
    want = B.forward_backward(parent, *seen, b, gh, np.zeros_like(gh))[2:]
    for name, a, r in zip(("dx", "dW", "dU", "db"), got, want):
        err = float(np.abs(a.cpu().numpy() - r).max() / max(1.0, np.abs(r).max()))
        assert err <= TOL[dtype], (name, err)
