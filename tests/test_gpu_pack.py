"""Weights of several cells packed in one launch, at widths that fill no 16-byte piece, no K step and no unit tile: every tree of
a typed table against the plain forward under its own cell's weights."""
import numpy as np
import pytest

from workloads import make_forest, tree_ranges
from gpu_util import dev_parent

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D,H", [(1, 1), (7, 5), (33, 31), (203, 99), (64, 32), (300, 260)])
def test_cells_packed_together(D, H, dtype):
    import torch
    import paper_1904_07421_amd as J
    p, n_sig = make_forest(1), 3
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(D + H)
    r = lambda *s: torch.rand(s, generator=g, device="cuda") - 0.5
    x, W, U, b = r(len(p), D).to(dt), r(n_sig, 4 * H, D).to(dt), (r(n_sig, 4 * H, H) * 0.3).to(dt), r(n_sig, 4 * H)
    cuts = tree_ranges(p)
    sig = np.zeros(len(p), dtype=np.int32)
    for t in range(len(cuts) - 1):
        sig[cuts[t]:cuts[t + 1]] = t % n_sig
    parent = dev_parent(p)
    st = J.jitdb_schedule_typed(parent, torch.from_numpy(sig).cuda(), n_sig)
    h, c = J.jitdb_treelstm_forward_typed(x, W, U, b, st)
    hp, cp = J.jitdb_treelstm_forward_packed(x, J.jitdb_treelstm_pack(W, U, b), st)
    assert torch.equal(h, hp) and torch.equal(c, cp)
    s = J.jitdb_schedule(parent)
    # two forms of the same sums: fp32 rounding, or (bf16) operands of eight bits passed up five levels
    tol = 1e-5 if dtype == "f32" else 2e-2
    for t in range(n_sig):
        h1, c1 = J.jitdb_treelstm_forward(x, W[t].contiguous(), U[t].contiguous(), b[t].contiguous(), s)
        rows = torch.from_numpy(sig == t).cuda()
        assert (h[rows].float() - h1[rows].float()).abs().max() <= tol and (c[rows] - c1[rows]).abs().max() <= tol
