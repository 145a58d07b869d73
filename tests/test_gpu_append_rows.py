"""Pool contents after appends, bit for bit: pieces that begin and end inside a
16-row group of the transposed V pool, cover whole groups, span 64-row chunks
and need several launches; and a prefill whose tables take several copying
workgroups.  Rows that no append wrote keep their bits."""

from __future__ import annotations

import numpy as np
import pytest

from tests.test_gpu_prefill import _Rig

pytestmark = pytest.mark.gpu

FILL = -1  # int16 bits the pools start with


def _pools(rig, rows):
    k = rig.kp.view(rig.hkv, rows, rig.d).cpu().view(__import__("torch").int16).numpy()
    v = rig.vp.view(rig.hkv, rows // 16, rig.d, 16).cpu().view(__import__("torch").int16).numpy()
    return k, v.transpose(0, 1, 3, 2).reshape(rig.hkv, rows, rig.d)


def _expect(rig, rows, writes):
    k = np.full((rig.hkv, rows, rig.d), FILL, np.int16)
    v = np.full((rig.hkv, rows, rig.d), FILL, np.int16)
    for at, ks, vs in writes:
        k[:, at] = ks.transpose(1, 0, 2)
        v[:, at] = vs.transpose(1, 0, 2)
    return k, v


def _random(rng, n, rig):
    return rng.integers(-30000, 30000, (2, n, rig.hkv, rig.d)).astype(np.int16)


@pytest.mark.parametrize("bt", [16, 64])
@pytest.mark.parametrize("d,hkv", [(64, 1), (128, 3)])
@pytest.mark.parametrize("counts", [(1, 7, 8, 9, 15, 16, 17), (16, 8, 8, 31, 64, 1), (129, 5, 66)])
def test_append_rows(counts, d, hkv, bt):
    print(f"[append rows counts={counts} d={d} hkv={hkv} B={bt}]", flush=True)
    rng = np.random.default_rng(1)
    blocks, n_nodes = 100 * 64 // bt, 5
    rig = _Rig(hkv, hkv, d, 1, num_blocks=blocks, bt=bt, live=True)
    nodes = [rig.ctx.new_root(200) for _ in range(n_nodes)]
    writes = []
    for step, c in enumerate(counts):
        ntok = [c if i != step % n_nodes else max(0, c - 1) for i in range(n_nodes)]  # lengths drift apart
        at = rig.ctx.kv_slots(nodes, ntok)
        kv = _random(rng, sum(ntok), rig)
        rig.ctx.kv_append(nodes, ntok, rig.dev(kv[0]), rig.dev(kv[1]))
        writes.append((at, kv[0], kv[1]))
    got, want = _pools(rig, blocks * bt), _expect(rig, blocks * bt, writes)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.parametrize("n", [1, 32, 33, 128, 256, 257, 300])
def test_one_token_steps(n):
    """One token per leaf at every place of a 16-row group; both batch sizes, several launches past 256 leaves."""
    print(f"[append steps n={n}]", flush=True)
    rng = np.random.default_rng(2)
    rig = _Rig(2, 2, 64, 1, num_blocks=n + 1, live=True)
    nodes = [rig.ctx.new_root(64) for _ in range(n)]
    writes = []
    for _ in range(18):
        at = rig.ctx.kv_slots(nodes, [1] * n)
        kv = _random(rng, n, rig)
        rig.ctx.kv_append(nodes, [1] * n, rig.dev(kv[0]), rig.dev(kv[1]))
        writes.append((at, kv[0], kv[1]))
    got, want = _pools(rig, (n + 1) * 64), _expect(rig, (n + 1) * 64, writes)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    assert (rig.node_len[:n].cpu().numpy() == 18).all()


def test_prefill_tables_over_several_copy_groups():
    """600 sequences: 19 KB of items and more of tiles; every row and length arrives."""
    print("[append prefill 600 sequences]", flush=True)
    n, blocks = 600, 1300
    rig = _Rig(2, 1, 64, 5, num_blocks=blocks, live=True)
    rng = np.random.default_rng(3)
    lens = [int(x) for x in rng.integers(1, 70, n)]
    roots = [rig.ctx.new_root(x) for x in lens]
    assert [rig.model.new_root(x) for x in lens] == roots
    at = rig.ctx.kv_slots(roots, lens)
    qb, out, lse = rig.prefill(roots, lens, 0)
    rig.check(roots, lens, qb, out, lse, "600 prompts", rows=np.arange(0, sum(lens), 37))
    ks = np.concatenate([rig.kv[r][0] for r in roots]).view(np.int16)
    vs = np.concatenate([rig.kv[r][1] for r in roots]).view(np.int16)
    got, want = _pools(rig, blocks * 64), _expect(rig, blocks * 64, [(at, ks, vs)])
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    assert rig.node_len[:n].cpu().tolist() == lens
