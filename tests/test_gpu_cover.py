"""Repairs and reverse edges decided from the covered pairs alone, against the oracle, bit for bit.

The rows run from tight clusters (few covered pairs, or none) to a few values
per byte in few dimensions (more covered pairs than the kernels take, repeated
vectors, ties of distance between different ids); degrees and prune caps end at
and inside the tiles of 16 slots; deletions are heavy enough for several deleted
neighbors per repaired node, and one batch of inserts lands in one cluster, so
that nodes get more offers than a batch of lanes holds.
"""

import numpy as np
import pytest

import oracle
from common import assert_same_state

pytestmark = pytest.mark.gpu


def rows(rng, n, dim, kind):
    if kind == "coarse":  # few values: repeated vectors and many equal distances
        return rng.integers(0, 3, (n, dim)).astype(np.uint8) * 100
    if kind == "uniform":
        return rng.integers(0, 256, (n, dim)).astype(np.uint8)
    c = np.random.default_rng(5).uniform(20, 235, (1 if kind == "one" else 6, dim))
    return np.clip(np.rint(c[rng.integers(0, c.shape[0], n)] + rng.standard_normal((n, dim)) * 18), 0, 255).astype(np.uint8)


@pytest.mark.parametrize("dim,R,cap,alpha,kind", [
    (128, 32, None, (6, 5), "clusters"), (128, 31, 32, (6, 5), "clusters"), (128, 17, 19, (1, 1), "clusters"),
    (128, 1, 4, (6, 5), "one"), (128, 32, None, (13, 10), "clusters"), (128, 16, None, (6, 5), "coarse"),
    (64, 32, 40, (6, 5), "uniform"), (64, 5, 9, (3, 1), "clusters"), (32, 24, None, (6, 5), "one"),
    (32, 32, 33, (6, 5), "coarse"), (16, 15, None, (1, 1), "coarse"), (16, 32, None, (6, 5), "uniform")])
def test_repairs_and_reverse_edges(dim, R, cap, alpha, kind):
    import torch
    from paper_2607_02543_amd import etale
    rng = np.random.default_rng(1000 * R + dim)
    kw = dict(alpha=alpha, n_entry=40, prune_cap=cap)
    slabs = 6000 + 500 * (R + 2)
    o = oracle.Oracle(oracle.METRIC_L2_U8, dim, R, 40, 2000, slabs, **kw)
    g = etale.Index(dim, R=R, L_build=40, id_capacity=2000, slab_capacity=slabs, max_batch=500, **kw)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    live, nxt = np.zeros(0, np.int64), 0

    def insert(n, kind):
        nonlocal live, nxt
        x = rows(rng, n, dim, kind)
        o.insert(x)
        g.insert(up(x))
        live = np.concatenate([live, np.arange(nxt, nxt + n)])
        nxt += n
        assert_same_state(o, g, f"{nxt} inserted")

    for n in (1, 70, 330):
        insert(n, kind)
    for r in range(3):
        dl = np.sort(rng.choice(live, len(live) // 5, replace=False)).astype(np.uint32)
        live = np.setdiff1d(live, dl)
        o.delete(dl)
        g.delete(up(dl.astype(np.int32)))
        assert_same_state(o, g, f"delete {r}")
        insert(200, "one" if r == 1 and kind == "clusters" else kind)  # lists still name the deleted ids
        if r != 1:  # a delete after this one meets older tombstones
            o.reclaim()
            g.reclaim()
            assert_same_state(o, g, f"reclaim {r}")
    g.close()


@pytest.mark.parametrize("n", [1, 255, 1000])
def test_delete_statuses(n):
    """Repeats, ids never handed out (repeated too) and ids already deleted, across workgroups."""
    import torch
    from paper_2607_02543_amd import etale
    rng = np.random.default_rng(n)
    o = oracle.Oracle(oracle.METRIC_L2_U8, 64, 12, 20, 1000, 30000, n_entry=16)
    g = etale.Index(64, R=12, L_build=20, id_capacity=1000, slab_capacity=30000, max_batch=1000, n_entry=16)
    for b in (100, 500):
        x = rows(rng, b, 64, "clusters")
        o.insert(x)
        g.insert(torch.from_numpy(x).cuda())
    for _ in range(3):
        ids = rng.integers(0, 600, n).astype(np.uint32)
        odd = rng.random(n)
        ids = np.where(odd < 0.1, rng.choice([600, 650, 999, 1000, 5000, 0xFFFFFFFE, 0xFFFFFFFF], n), ids).astype(np.uint32)
        ids = np.where(odd > 0.8, ids[rng.integers(0, n, n)], ids)
        so = o.delete(ids)
        sg = g.delete(torch.from_numpy(ids.astype(np.int64).astype(np.uint32).view(np.int32)).cuda()).cpu().numpy()
        assert np.array_equal(so, sg)
        assert_same_state(o, g, "after the deletes")
    g.close()
