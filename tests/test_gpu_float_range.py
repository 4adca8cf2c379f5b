"""Float rows and queries at the ends of binary32's range: results depend neither on a power of two moved from the
queries to the rows nor on the path that computes a distance."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _up(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# rows shared by 2 and by 16 lanes (one reduction each). Components of size 2^-122 keep all 24 bits: their products with
# a code's value / 256 (of [0.875, 1.75], in steps of 2^-4) are whole multiples of the smallest subnormal
@pytest.mark.parametrize("dim", [96, 768])
def test_fp8_queries_near_the_smallest_normal(dim):
    from paper_2607_02543_amd import etale
    rng = np.random.default_rng(dim)
    n, R = 200, 16
    x = (rng.uniform(0.5, 1, (n, dim)) * rng.choice([-1, 1], (n, dim))).astype(np.float32)
    q = (rng.uniform(0.5, 1, (40, dim)) * rng.choice([-1, 1], (40, dim))).astype(np.float32)
    nbr = np.array([rng.choice(np.delete(np.arange(n), i), R, replace=False) for i in range(n)], np.uint32)
    found = []
    for e in (0, 121):
        g = etale.Index(dim, R=R, L_build=32, n_entry=1, id_capacity=256, slab_capacity=20_000, max_batch=n,
                        metric=etale.METRIC_IP_F32, traversal=etale.TRAV_FP8, rerank_mult=0, W=1)
        g.insert(_up(np.ldexp(x, e - 4)))
        g.set_lists(np.arange(n), nbr, np.full(n, R))  # the same graph for both, whatever its distances
        i, d = g.search(_up(np.ldexp(q, -e)), 10, 64)
        found.append((i.cpu().numpy(), d.cpu().numpy()))
        g.close()
    assert np.array_equal(found[0][0], found[1][0])
    assert np.array_equal(found[0][1], found[1][1])


def _strange(rng, n, dim):
    """Unit rows; in two fifths of them one component, in a few of them all, an infinity or a NaN of either sign."""
    x = rng.standard_normal((n, dim)).astype(np.float32)
    x /= np.linalg.norm(x, axis=1, keepdims=True)
    odd = np.array([0x7F800000, 0xFF800000, 0x7FC00000, 0xFFC00000], np.uint32).view(np.float32)
    for i in np.flatnonzero(rng.random(n) < 0.4):
        x[i, rng.integers(0, dim, rng.integers(1, 3))] = odd[rng.integers(0, 4)]
    for j, i in enumerate(rng.choice(n, 8, replace=False)):
        x[i] = odd[j % 4]
    return x


def _distances(x, q):
    """q's distances to each row of x as the brute force gives them when that row is among sixteen live ones."""
    from paper_2607_02543_amd import etale
    g = etale.Index(x.shape[1], R=4, L_build=8, n_entry=16, id_capacity=x.shape[0], slab_capacity=4000, max_batch=16,
                    metric=etale.METRIC_IP_F32)
    out = np.empty((q.shape[0], x.shape[0]), np.uint32)
    for b in range(0, x.shape[0], 16):
        at = g.insert(_up(x[b:b + 16]))
        i, d = g.bruteforce(_up(q), at.numel())
        i, d = i.cpu().numpy(), d.cpu().numpy().view(np.uint32)
        assert np.array_equal(np.sort(i, axis=1), np.tile(at.cpu().numpy(), (q.shape[0], 1)))
        np.put_along_axis(out, i, d, axis=1)
        g.delete(at)
        g.reclaim()
    g.close()
    return out


# the first pass's order of a sum need not be the second's where a NaN is in it: groups of 64 rows with and without one
@pytest.mark.parametrize("dim", [96, 192, 384, 768])
def test_infinities_and_nans_rank_by_the_rows_own_distance(dim):
    from paper_2607_02543_amd import etale
    rng = np.random.default_rng(dim + 1)
    n = 960
    x, q = _strange(rng, n, dim), _strange(rng, 50, dim)
    x[320:640] = np.abs(np.nan_to_num(x[320:640], nan=0.0, posinf=0.0, neginf=0.0))
    d = _distances(x, q)
    g = etale.Index(dim, R=12, L_build=16, n_entry=100, id_capacity=n, slab_capacity=20_000, max_batch=240,
                    metric=etale.METRIC_IP_F32)
    for b in range(0, n, 240):
        g.insert(_up(x[b:b + 240]))
    i, got = g.bruteforce(_up(q), 16)
    i, got = i.cpu().numpy(), got.cpu().numpy().view(np.uint32)
    key = np.where(d >> 31, ~d, d | 0x80000000).astype(np.uint32)  # the order of binary32 values, NaNs at both ends
    want = np.stack([np.lexsort((np.arange(n), r))[:16] for r in key])
    assert np.array_equal(got, np.take_along_axis(d, want, axis=1))
    assert np.array_equal(i, want)
    g.close()


# with every row in the entry set a search starts from its exact nearest rows: tiles of three sizes, the selection from
# registers, from group minima and the general one. Values in eighths, so that every finite sum is exact
@pytest.mark.parametrize("dim,n,nq", [(96, 700, 20), (96, 4200, 1100), (192, 260, 300), (768, 300, 33)])
def test_start_lists_with_infinities_and_nans(dim, n, nq):
    from paper_2607_02543_amd import etale
    rng = np.random.default_rng(n + dim)
    x = (rng.integers(-2, 3, (n, dim)) / 8).astype(np.float32)
    q = (rng.integers(-2, 3, (nq, dim)) / 8).astype(np.float32)
    q[q == 0] = 0.125
    for v in (np.inf, -np.inf, np.nan):
        at = rng.choice(n, 8, replace=False)
        x[at, rng.integers(0, dim, 8)] = v
    q[3, 5], q[4, 6] = np.inf, -np.inf
    g = etale.Index(dim, R=8, L_build=16, n_entry=n, id_capacity=n, slab_capacity=30 * n, max_batch=n, metric=etale.METRIC_IP_F32)
    g.insert(_up(x))
    with np.errstate(invalid="ignore"):
        d = (1 - np.stack([(x.astype(np.float64) * r.astype(np.float64)).sum(1) for r in q])).astype(np.float32)
    # a row's own NaN is positive and its distance negative: before every other. A NaN of the hardware's own making (an
    # infinite component of the query on a zero) is negative and its distance positive: after every other
    own = np.isnan(x).any(1)
    place = np.where(own[None, :], 0, np.where(np.isnan(d), 2, 1))
    want = np.stack([np.lexsort((np.arange(n), np.nan_to_num(r, nan=0.0, posinf=np.inf, neginf=-np.inf), c))[:10]
                     for r, c in zip(d, place)])
    for L in (16, 64, 128, 200):
        i, got = g.search(_up(q), 10, L)
        assert np.array_equal(i.cpu().numpy(), want), L
        assert np.array_equal(got.cpu().numpy(), np.take_along_axis(d, want, axis=1), equal_nan=True), L
    finite = np.isfinite(q).all(1)  # with both kinds of NaN in a row's sum its lanes' order decides
    i, got = g.bruteforce(_up(q[finite]), 10)
    assert np.array_equal(i.cpu().numpy(), want[finite])
    g.close()
