"""Workspaces: what their sizes promise, worked out on the host (no GPU)."""
import ctypes

import numpy as np
import pytest

import paper_1904_07421_amd as J
from paper_1904_07421_amd import binding


def _up(a, b):
    return -(-a // b) * b


def _needed(n, leaves, D, H, esz):
    """Bytes of the operands by node and of the partial sums as the launch cuts them (128 x 256 tiles of fp32 a range)."""
    Hk, rows = _up(H, 64), _up(n, 64)
    n4, mx, mh = Hk // 64, -(-(D + 1) // 128), -(-H // 128)
    tiles = mx * n4, mh * -(-3 * Hk // 256), mh * -(-Hk // 256)
    f = mx * (n4 - 3 * Hk // 256) if 3 * Hk % 256 == 0 else 0        # tiles with nothing but the forget gate
    work = (tiles[0] - f + tiles[2]) * rows + (tiles[1] + f) * (rows - leaves // 64 * 64)
    per = _up(-(-work // 512), 64)
    if per >= 16384:
        per = _up(per // 8, 64)
    splits = -(-rows // min(max(per, 128), rows))
    operands = n * (4 * H + esz * (H + _up(4 * Hk, 256) + _up(Hk, 256) + _up(D + 1, 128) + 2 * _up(H, 128)))
    return operands + splits * sum(tiles) * 128 * 256 * 4


def _bytes(n, leaves, D, H, dtype):
    levels = np.array([0, leaves, n], dtype=np.int32)
    s = binding._ScheduleStruct(n_nodes=n, host_level_ptr=levels.ctypes.data, n_levels=2)
    lib = binding.load_library()
    return int(lib.jitdb_treelstm_backward_workspace_bytes(ctypes.byref(s), D, H, dtype))


@pytest.mark.parametrize("D,H", [(300, 150), (300, 512), (64, 1024), (24, 24), (300, 4096)])
def test_partial_sums_have_room_whatever_the_leaves(D, H):
    for n in (1, 64, 1000, 6000, 70000, 250000, 650000, 3000000):
        for share in (0.02, 0.25, 0.5, 0.75, 1.0):
            leaves = max(1, int(n * share))
            if leaves < n:
                got = _bytes(n, leaves, D, H, J.JITDB_BF16)
                assert got >= _needed(n, leaves, D, H, 2), (n, leaves, D, H)


@pytest.mark.parametrize("D,H,dtype", [(24, 24, J.JITDB_F32), (300, 150, J.JITDB_BF16), (300, 256, J.JITDB_F32), (300, 512, J.JITDB_BF16)])
def test_a_larger_forests_workspace_holds_a_smaller_ones(D, H, dtype):
    sizes = [1, 1000, 65536, 65537, 262143, 262144, 262145, 300000, 600000, 2000000]
    for n_sig in (1, 3):
        forward = [J.jitdb_treelstm_typed_workspace_bytes(n, n - 1, D, H, dtype, n_sig) for n in sizes]
        assert forward == sorted(forward), (n_sig, forward)
    cells = [J.jitdb_treelstm_cells_workspace_bytes(n, n - 1, D, H, dtype, [(J.JITDB_CELL_NARY, 2)]) for n in sizes]
    assert cells == sorted(cells)
    backward = [_bytes(n, max(1, n // 2), D, H, dtype) for n in sizes[1:]]
    assert backward == sorted(backward)


@pytest.mark.parametrize("D,H,dtype,n,plain", [(300, 256, J.JITDB_BF16, 300000, True), (300, 150, J.JITDB_F32, 200000, False),
                                               (700, 256, J.JITDB_BF16, 60000, True)])
def test_no_room_for_whole_trees_where_they_do_not_run(D, H, dtype, n, plain):
    """Past the largest forest that runs as whole trees, in tables of several cells and where D or H rule them out, a
    workspace is what its nodes and its weights take.  The nodes' part is what it grows by from there."""
    asks = [lambda m: J.jitdb_treelstm_typed_workspace_bytes(m, m - 1, D, H, dtype, 3),
            lambda m: J.jitdb_treelstm_cells_workspace_bytes(m, m - 1, D, H, dtype, [(J.JITDB_CELL_NARY, 2)])]
    if plain:
        asks.append(lambda m: J.jitdb_treelstm_workspace_bytes(m, m - 1, D, H, dtype))
    for ask in asks:
        per_node = (ask(9 * n) - ask(8 * n)) / n
        weights = 8 * 4 * 512 * (_up(D, 64) + 3 * 256 + 64) * 4           # generous: every cell padded to 512 units, fp32
        assert ask(n) <= n * per_node + weights + (1 << 20), (ask(n), n * per_node)


@pytest.mark.parametrize("H", [161, 168, 176, 177, 192, 193, 208, 224, 240, 256])
@pytest.mark.parametrize("D", [1, 64, 65, 127, 128, 192, 255, 256, 300, 512, 640])
def test_wide_cells_ask_300_000_nodes_for_their_levels_alone(D, H):
    """bf16 cells of more than 160 units: from there on the plain forward asks for what a table of one such cell takes (that of
    two cells without the second cell's weights), which never has room for whole trees."""
    for n in (300000, 450000, 1000000):
        two, three = (J.jitdb_treelstm_typed_workspace_bytes(n, n - 1, D, H, J.JITDB_BF16, k) for k in (2, 3))
        assert J.jitdb_treelstm_workspace_bytes(n, n - 1, D, H, J.JITDB_BF16) <= 2 * two - three + 256, (n, D, H)
    sizes = [1, 1000, 65536, 65537, 81920, 81921, 100000, 110000, 120000, 262144, 262145, 300000, 600000]
    asked = [J.jitdb_treelstm_workspace_bytes(n, n - 1, D, H, J.JITDB_BF16) for n in sizes]
    assert asked == sorted(asked)
