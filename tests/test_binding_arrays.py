"""Array arguments of the binding: writable, read-only, empty, strided and
converted arrays give the library the same ids; repeated and unordered nodes
in one append keep their rows."""

import numpy as np
import pytest

from paper_2508_17445_amd.treepo import TreePOError
from tests.lib_helpers import host_ctx


def _forms(xs):
    a = np.array(xs, np.int32)
    ro = a.copy()
    ro.flags.writeable = False
    return [list(xs), tuple(xs), a, ro, a.astype(np.int64), np.repeat(a, 2)[::2], a.reshape(1, -1)]


def test_every_array_form():
    want = None
    for k in range(7):
        ctx = host_ctx()
        r = [ctx.new_root(200) for _ in range(3)]
        nodes = _forms([r[2], r[0], r[2]])[k]  # unordered, repeated
        ntok = _forms([70, 1, 5])[k]
        rows = ctx.kv_slots(nodes, ntok)
        ctx.kv_commit(nodes, ntok)
        got = (rows.tolist(), ctx.export_nodes().tolist(), ctx.workspace_size(_forms([r[0], r[2]])[k]))
        want = want or got
        assert got == want
    assert want[1][2][3] == 75 and want[1][0][3] == 1


def test_empty_arrays():
    ctx = host_ctx()
    ctx.new_root(10)
    ctx.kv_commit(np.zeros(0, np.int32), [])
    with pytest.raises(TreePOError):
        ctx.workspace_size(np.zeros(0, np.int32))


def test_repeated_nodes_fill_up():
    """The lengths of a repeated node add up, ascending or not."""
    for order in ([0, 0, 1], [1, 0, 0], [0, 1, 0]):
        ctx = host_ctx()
        r = [ctx.new_root(10), ctx.new_root(10)]
        with pytest.raises(TreePOError):
            ctx.kv_commit([r[i] for i in order], [6 if i == 0 else 1 for i in order])
        ctx.kv_commit([r[i] for i in order], [5 if i == 0 else 1 for i in order])
        assert ctx.export_nodes()[:, 3].tolist() == [10, 1]
