"""Float rows whose distances FP32 holds exactly, so GPU and oracle must agree with no tolerance.

Every row has a fixed number of entries of one size, 7/8 of a power of two, and
either sign, the rest zero: products and partial sums are multiples of that size
squared and stay far below 2^24 of them, so FP32 sums in any order equal the
FP64 oracle's. The bf16 copy holds such rows exactly, and so does the FP8 copy
(its scale, the size over 448, is a power of two). The rows come in clusters (a center with a few signs turned), so
prunes cover candidates, and distances take few values, so ties are common and
the order by id decides them.
"""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def lattice(rng, n, dim, centers=12, turn=0.08):
    """n rows of 4^j entries of size 7/8 2^-j, exact in FP32, bf16 and scaled FP8."""
    j = {96: 3, 192: 3, 384: 4, 768: 4}[dim]
    nz = 4 ** j
    c = np.zeros((centers, dim), np.float32)
    for r in c:
        at = rng.permutation(dim)[:nz]
        r[at] = rng.choice([-1.0, 1.0], nz)
    x = c[rng.integers(0, centers, n)]
    x = np.where(rng.random(x.shape) < turn, -x, x)
    return (x * 0.875 * 2.0 ** -j).astype(np.float32)


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


# a step's rows are gathered eight per lane group at a time (fewer where fewer
# than eight lanes share a row): batches inside, at and past that, for every
# copy, with one, two and four expansions per step and both list forms
@pytest.mark.parametrize("trav", [0, 1, 2])
@pytest.mark.parametrize("dim,R,W", [(96, 7, 1), (96, 32, 2), (96, 32, 4), (192, 20, 2), (384, 24, 1), (768, 48, 1)])
def test_searches_equal_oracle(dim, R, W, trav):
    import torch
    # rerank 0: the traversal's own distances (in FP32 traversal there is no re-rank)
    o, g, rng = churned_pair(dim, R, 7 * R + dim + trav, rounds=1, W=W, traversal=trav, rerank_mult=0)
    q = lattice(rng, 70, dim)
    qd = torch.from_numpy(q).cuda()
    for k, L in ((10, 16), (5, 64), (10, 100), (60, 128), (20, 200)):
        io, do, eo, no = o.search(q, k, L, counts=True)
        ig, dg, cg = g.search(qd, k, L, counts=True)
        assert np.array_equal(io, ig.cpu().numpy().astype(np.uint32)), (k, L)
        assert np.array_equal(do, dg.cpu().numpy().astype(np.float64)), (k, L)
        assert np.array_equal(eo, cg[:, 0].cpu().numpy().astype(np.uint32)), (k, L)
    g.close()


def test_fp8_nan_codes_keep_their_value():
    """A row with a NaN component has the code 0x7F there, which every FP8 traversal reads as 480 (times the scale)."""
    import torch
    from paper_2607_02543_amd import etale
    rng = np.random.default_rng(3)
    x = lattice(rng, 40, 96)
    x[5:20, 3] = np.nan
    x[9, 50:53] = np.nan
    g = etale.Index(96, R=32, L_build=64, n_entry=1, id_capacity=64, slab_capacity=4000, max_batch=40,
                    metric=etale.METRIC_IP_F32, traversal=etale.TRAV_FP8, rerank_mult=0)
    g.insert(torch.from_numpy(x).cuda())
    nbr = np.full((1, 32), 0, np.uint32)
    nbr[0, :30] = np.arange(1, 31)
    g.set_lists([0], nbr, [30])
    codes, s = g.rows(0, 40, 2), g.rows(0, 40, 3).astype(np.float64)
    assert (codes[5:20, 3] == 0x7F).all()
    v = np.where(codes & 0x80, -1.0, 1.0)
    e, m = (codes >> 3) & 15, codes & 7
    v = v * np.where(e == 0, m * 2.0 ** -9, (8 + m) * 2.0 ** (e.astype(np.float64) - 10))
    q = lattice(rng, 8, 96)
    ids, d = g.search(torch.from_numpy(q).cuda(), 31, 64)
    ids, d = ids.cpu().numpy(), d.cpu().numpy().astype(np.float64)
    for i in range(q.shape[0]):
        assert np.isfinite(d[i]).all()
        assert np.array_equal(d[i], 1.0 - (v[ids[i]] @ q[i].astype(np.float64)) * s[ids[i]])
    g.close()


# groups of 64 rows, 16 queries per wave and 64 per workgroup: counts inside, at
# and past them, with deleted rows, fewer live rows than asked for, and none
@pytest.mark.parametrize("dim,n,nq", [(96, 63, 1), (96, 700, 65), (192, 64, 16), (384, 65, 17), (768, 300, 130)])
def test_bruteforce_equals_oracle(dim, n, nq):
    import torch
    rng = np.random.default_rng(n + dim)
    o, g = make_pair(dim, 8)
    q = lattice(rng, nq, dim)
    qd = torch.from_numpy(q).cuda()

    def check(k):
        io, do = o.bruteforce(q, k)
        ig, dg = g.bruteforce(qd, k)
        assert np.array_equal(io, ig.cpu().numpy().astype(np.uint32))
        assert np.array_equal(do, dg.cpu().numpy().astype(np.float64))

    for b in range(0, n, 400):
        x = lattice(rng, min(400, n - b), dim)
        o.insert(x)
        g.insert(torch.from_numpy(x).cuda())
    for k in (1, 10, 16):
        check(k)
    for gone in (np.arange(0, n, 3), np.setdiff1d(np.arange(n), np.concatenate([np.arange(0, n, 3), [1, n - 1]]))):
        for c in range(0, gone.size, 400):
            o.delete(gone[c:c + 400].astype(np.uint32))
            g.delete(torch.from_numpy(gone[c:c + 400].astype(np.int32)).cuda())
        check(10)
    g.close()
