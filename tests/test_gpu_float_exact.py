"""Float rows whose distances FP32 holds exactly, so GPU and oracle must agree with no tolerance.

Every row has a fixed number of entries of one power-of-two size and either
sign, the rest zero: products and partial sums are multiples of that size
squared and stay far below 2^24 of them, so FP32 sums in any order equal the
FP64 oracle's. The rows come in clusters (a center with a few signs turned), so
prunes cover candidates, and distances take few values, so ties are common and
the order by id decides them.
"""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def lattice(rng, n, dim, centers=12, turn=0.08):
    """n rows of 4^j entries of size 2^-j: unit norm, exact in FP32."""
    j = {96: 3, 192: 3, 384: 4, 768: 4}[dim]
    nz = 4 ** j
    c = np.zeros((centers, dim), np.float32)
    for r in c:
        at = rng.permutation(dim)[:nz]
        r[at] = rng.choice([-1.0, 1.0], nz)
    x = c[rng.integers(0, centers, n)]
    x = np.where(rng.random(x.shape) < turn, -x, x)
    return (x * 2.0 ** -j).astype(np.float32)


def make_pair(dim, R, L_build=40, n_entry=50, prune_cap=None, W=1, cap=2000, max_batch=400, **kw):
    from paper_2607_02543_amd import etale
    slabs = 3 * cap + max_batch * (R + 2)
    o = oracle.Oracle(oracle.METRIC_IP_F32, dim, R, L_build, cap, slabs, n_entry=n_entry, prune_cap=prune_cap, W=W, **kw)
    g = etale.Index(dim, R=R, L_build=L_build, n_entry=n_entry, id_capacity=cap, slab_capacity=slabs,
                    max_batch=max_batch, metric=etale.METRIC_IP_F32, prune_cap=prune_cap, W=W, **kw)
    return o, g


def assert_equal_state(o, g, where):
    eo, eg = o.export(), g.export()
    for f in ("deg", "deleted", "has_slab", "nbr"):
        assert np.array_equal(eo[f], eg[f]), f"{where}: {f}"
    assert np.array_equal(eo["rho"].astype(np.float64), eg["rho"].astype(np.float64)), f"{where}: distances"
    mo, sg = eo["meta"], g.stats()
    assert sg["error_bits"] == 0
    for a, b in (("free", "free_slabs"), ("resident", "resident_slabs")):
        assert mo[a] == sg[b], f"{where}: {a}"
    for k in ("pub_forward", "pub_repair", "pub_reverse", "pub_refine", "pub_compact", "freed"):
        assert mo[k] == sg[k], f"{where}: {k}"


def churned_pair(dim, R, seed, rounds=2, **kw):
    import torch
    rng = np.random.default_rng(seed)
    o, g = make_pair(dim, R, **kw)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    live = np.zeros(0, np.int64)
    nxt = 0
    for b in (60, 150, 240):
        x = lattice(rng, b, dim)
        o.insert(x)
        g.insert(up(x))
        live = np.concatenate([live, np.arange(nxt, nxt + b)])
        nxt += b
        assert_equal_state(o, g, f"after {nxt} inserts")
    for r in range(rounds):
        dl = np.sort(rng.choice(live, 60, replace=False)).astype(np.uint32)
        live = np.setdiff1d(live, dl)
        o.delete(dl)
        g.delete(up(dl.astype(np.int32)))
        assert_equal_state(o, g, f"delete {r}")
        x = lattice(rng, 70, dim)
        o.insert(x)
        g.insert(up(x))
        live = np.concatenate([live, np.arange(nxt, nxt + 70)])
        nxt += 70
        assert_equal_state(o, g, f"insert {r}")
        o.reclaim()
        g.reclaim()
        assert_equal_state(o, g, f"reclaim {r}")
    return o, g, rng


# prunes decide their candidates in blocks of eight over rows shared by 8, 16,
# 32 or 64 lanes: degrees and caps that end inside, at and past a block
@pytest.mark.parametrize("dim,R,cap", [(96, 1, 8), (96, 7, 15), (96, 32, None), (192, 8, 17), (192, 33, 40),
                                       (384, 12, 12), (384, 24, None), (768, 9, 64), (768, 48, 98)])
def test_maintenance_equals_oracle(dim, R, cap):
    o, g, _ = churned_pair(dim, R, 100 * R + dim, prune_cap=cap)
    g.close()
