"""Row records of levels that run one by one (forward.hip): forests smaller than a record's four child ids, child lists that end with
the CSR, and windows full and short, against the C oracle."""
import numpy as np
import pytest

from workloads import make_forest, make_values, chain_forest, star_forest
from gpu_util import run_gpu_forward

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


def _lay_out(trees):
    off = np.concatenate([[0], np.cumsum([t.shape[0] for t in trees])])
    return np.concatenate([np.where(t < 0, -1, t + o) for t, o in zip(trees, off)]).astype(np.int32)


FORESTS = {
    "one": lambda: np.array([-1], dtype=np.int32),
    "two": lambda: chain_forest(2),
    "three": lambda: star_forest(2),
    "four": lambda: star_forest(3),
    "last-has-five": lambda: _lay_out([chain_forest(3), star_forest(5)]),
    "last-has-one": lambda: _lay_out([star_forest(6), chain_forest(2)]),
    "window": lambda: _lay_out([star_forest(3)] * 1024),                       # 4096 nodes
    "window-and-one": lambda: _lay_out([star_forest(3)] * 1024 + [chain_forest(1)]),
    "windows": lambda: _lay_out([make_forest(1)] * 120 + [star_forest(70)]),
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(FORESTS))
def test_records(c_oracle, name, dtype):
    p = FORESTS[name]()
    x, W, U, b = make_values(1, p.shape[0], "random", D=20, H=260)        # wider than whole trees go
    print(f"{name} {dtype} N={p.shape[0]}", flush=True)
    s, h, c, seen = run_gpu_forward(p, x, W, U, b, dtype)
    ho, co, _ = c_oracle(p, *seen)
    assert np.abs(h - ho).max() <= TOL[dtype]
    assert np.abs(c - co).max() <= TOL[dtype] * max(1.0, np.abs(co).max() / (8.0 if dtype == "bf16" else 50.0))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_training_forward_takes_other_windows(dtype):
    """From 262 144 nodes on the training forward orders its rows in larger windows than the forward."""
    import torch
    import paper_1904_07421_amd as J
    from gpu_util import dev_parent
    p = _lay_out([star_forest(2 + 7 * i % 23) for i in range(20300)] + [chain_forest(3)])
    assert 262144 < p.shape[0] < 300000
    D, H, dt = 20, 260, torch.float32 if dtype == "f32" else torch.bfloat16       # wider than whole trees go
    g = torch.Generator(device="cuda").manual_seed(7)
    r = lambda *s: torch.rand(s, generator=g, device="cuda") - 0.5
    x, W, U, b = r(len(p), D).to(dt), r(4 * H, D).to(dt), (r(4 * H, H) * 0.3).to(dt), r(4 * H)
    s = J.jitdb_schedule(dev_parent(p))
    h, c = J.jitdb_treelstm_forward(x, W, U, b, s)
    ht, ct, gates, fgate = J.jitdb_treelstm_forward_train(x, W, U, b, s)
    # two forms of the same sums (the training forward has no chain levels, and other levels are thin): 24-bit sums of up to 280 products of at
    # most 1/4, or (bf16) operands of eight bits; c adds up to 23 children
    tol = 2e-5 if dtype == "f32" else 2e-2
    assert (h.float() - ht.float()).abs().max() <= tol and (c - ct).abs().max() <= tol * max(1.0, float(c.abs().max()))
