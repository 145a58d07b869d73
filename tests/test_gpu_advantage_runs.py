"""GPU parity of the advantage kernel where its work is split: sub-groups
around the size one thread sums, one tree whose root holds every position,
and batches at and past the sizes that are staged in LDS (4,096 positions or
runs).  Bar as in the other advantage tests: 1e-6 against the fp64 oracle."""

from __future__ import annotations

import numpy as np
import pytest

from oracle import advantage as ADV
from tests.lib_helpers import host_ctx
from tests.test_gpu_advantage import TOL, _gpu_adv

pytestmark = pytest.mark.gpu


def _forest(groups, tail):
    """Per group size w: a root with w children, each under a chain of `tail` nodes."""
    ctx, parents, leaves = host_ctx(), [], []

    def grow(p, n):
        got = ctx.fork(p, n, 64) if p >= 0 else [ctx.new_root(64)]
        parents.extend([p] * len(got))
        return got

    for w in groups:
        root = grow(-1, 1)[0]
        for c in grow(root, w):
            for _ in range(tail):
                c = grow(c, 1)[0]
            leaves.append(c)
    return ctx, parents, leaves


@pytest.mark.parametrize("groups,tail", [
    ((1, 2, 15, 16, 17, 63, 64, 65), 2),
    ((1000,), 1),
    ((16,) * 240, 0),        # 3,840 positions, 4,080 runs: within the LDS sizes
    ((16,) * 241, 0),        # 4,097 runs
    ((4096,), 0),            # 4,096 positions, 4,097 runs
    ((700, 5000), 0),
])
def test_sizes(groups, tail):
    ctx, parents, leaves = _forest(groups, tail)
    rng = np.random.default_rng(len(leaves))
    perm = rng.permutation(len(leaves))
    lv = [leaves[i] for i in perm]
    for kind, rew in (("0/1", rng.integers(0, 2, size=len(lv))), ("normal", rng.normal(size=len(lv)))):
        rew = rew.astype(np.float32)
        for w, name in ((0, "mean"), (1, "size")):
            print(f"[advantage runs {groups[:3]} n={len(lv)} {kind} {name}]", flush=True)
            got = _gpu_adv(ctx, lv, rew, w)
            want = ADV.tree_advantage(parents, lv, rew.astype(np.float64), name)
            assert float(np.abs(got - want).max()) <= TOL
