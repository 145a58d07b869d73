"""Plans of one round at head dim 64 use three workgroups of a compute unit from
24 cost units per two-workgroup stream on, two below; head dim 128 always two.
Every chain token is covered once on both sides."""

import pytest

from tests.lib_helpers import host_ctx, oracle_model, replay_host
from tests.oracle_pins import _Log
from tests.test_metadata import _plan_checks, _stream_costs


@pytest.mark.parametrize("d,per_stream,slots", [(64, 20, 512), (64, 23, 512), (64, 26, 768), (64, 120, 768),
                                                (128, 20, 512), (128, 60, 512)])
def test_streams_by_cost(d, per_stream, slots):
    tokens = 32 * 512 * per_stream // 4
    n, cap = 4, 512
    ops = [("root", tokens), ("append", [0], [tokens]), ("fork", 0, n, cap),
           ("append", list(range(1, n + 1)), [65 + i for i in range(n)])]
    log = _Log(ops, list(range(1, n + 1)), {0: tokens, **{1 + i: 65 + i for i in range(n)}})
    ctx = host_ctx(hq=16, hkv=4, d=d)
    replay_host(ctx, log)
    pieces, tiles, n_streams = _plan_checks(ctx, oracle_model(log), log.leaves, 0)
    cost = _stream_costs(pieces, n_streams)
    assert (cost.sum() >= 24 * 512) == (slots == 768) or d == 128
    assert 0.95 * slots <= n_streams <= slots


def test_several_rounds_as_before():
    """Work past two workgroups' tables (192 cost units each) takes several
    rounds of short streams at D = 64 too, although three would hold it."""
    tokens = 32 * 512 * 220 // 4
    n = 4
    ops = [("root", tokens), ("append", [0], [tokens]), ("fork", 0, n, 64), ("append", [1, 2, 3, 4], [7] * n)]
    log = _Log(ops, [1, 2, 3, 4], {0: tokens, **{1 + i: 7 for i in range(n)}})
    ctx = host_ctx(hq=16, hkv=4, d=64)
    replay_host(ctx, log)
    pieces, _, n_streams = _plan_checks(ctx, oracle_model(log), log.leaves, 0)
    assert 192 * 512 < _stream_costs(pieces, n_streams).sum() < 192 * 768
    assert n_streams > 768


@pytest.mark.parametrize("n,slots", [(4, 768), (50, 512)])
def test_scratch_limit_keeps_two(n, slots):
    """One very long leaf cut over every stream sets the slot stride of all
    keys: where three workgroups' entries would pass the 64 MiB of the no-alloc
    scratch, the plan keeps two."""
    big = 32 * 512 * 30
    ctx = host_ctx(hq=8, hkv=1, d=64)
    r = ctx.new_root(64)
    ctx.kv_commit([r], [64])
    long_leaf, = ctx.fork(r, 1, big)
    kids = [long_leaf] + ctx.fork(r, n - 1, 64)
    ctx.kv_commit(kids, [big] + [5] * (n - 1))
    _, _, _, n_streams = ctx.export_plan(kids)
    assert 0.95 * slots <= n_streams <= slots
    assert ctx.workspace_size(kids) < 64 << 20
