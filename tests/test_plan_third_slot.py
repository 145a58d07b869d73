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
