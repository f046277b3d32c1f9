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
