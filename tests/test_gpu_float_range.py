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
