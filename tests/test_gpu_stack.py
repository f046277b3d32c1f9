"""Stack steps (forward.hip, cells.hip): rows around the 32 of a block and the 256 of the blocks that the XCDs take in turn, widths around
the 128 bytes of K that a block writes, rows of x on any element boundary, long child lists; against the oracles."""
import numpy as np
import pytest

from workloads import make_values, star_forest
from gpu_util import run_gpu_forward
from test_gpu_cells import _check

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


def _stars(roots, kids):
    """`roots` stars side by side, star i with 1 + i % kids leaves: two levels of known size."""
    parts, at = [], 0
    for i in range(roots):
        p = star_forest(2 + i % kids)
        parts.append(np.where(p < 0, -1, p + at))
        at += p.shape[0]
    return np.concatenate(parts).astype(np.int32)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("roots,kids,D,H", [(1, 1, 1, 257), (31, 3, 64, 257), (32, 9, 3, 258), (33, 5, 300, 257), (63, 6, 31, 257), (64, 4, 32, 260), (65, 7, 33, 264), (255, 4, 65, 260), (256, 5, 37, 264), (257, 6, 33, 257), (511, 2, 63, 257),
                                            (512, 3, 64, 257), (513, 5, 65, 320), (700, 9, 203, 260)])
def test_stack(c_oracle, roots, kids, D, H, dtype):
    p = _stars(roots, kids)
    x, W, U, b = make_values(1, p.shape[0], "random", D=D, H=H)        # wider than whole trees go
    print(f"stack {dtype} N={p.shape[0]} D={D} H={H}", flush=True)
    s, h, c, seen = run_gpu_forward(p, x, W, U, b, dtype)
    ho, co, _ = c_oracle(p, *seen)
    assert np.abs(h - ho).max() <= TOL[dtype]
    assert np.abs(c - co).max() <= TOL[dtype] * max(1.0, np.abs(co).max() / (8.0 if dtype == "bf16" else 50.0))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("roots,N,D,H", [(1, 1, 1, 1), (33, 3, 64, 32), (64, 2, 32, 33), (65, 3, 65, 31), (255, 2, 33, 40), (257, 4, 31, 33), (513, 4, 203, 64)])
def test_stack_of_nary_cells(roots, N, D, H, dtype):
    p = _stars(roots, N)
    _check(p, np.zeros(p.shape[0], np.int32), [N], D, H, dtype, 5)
