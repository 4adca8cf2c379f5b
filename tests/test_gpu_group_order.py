"""Nodes that many pairs of one phase are aimed at: hubs with runs of every length that the ordering of a target's
sources tells apart (4 | 64 | 128 | 256 | 512 pairs, pieces of 4,096), offered by one batch of inserts and then repaired
after one batch of deletes in no order, against the oracle."""

import time

import numpy as np
import pytest

import oracle
from common import assert_same_state

pytestmark = pytest.mark.gpu

DIM, R = 16, 6


def _up(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _pair(cap, batch, **kw):
    from paper_2607_02543_amd import etale
    slabs = 3 * cap + 2 * batch * (R + 2)
    o = oracle.Oracle(oracle.METRIC_L2_U8, DIM, R, 12, cap, slabs, n_entry=12, **kw)
    g = etale.Index(DIM, R=R, L_build=12, n_entry=12, id_capacity=cap, slab_capacity=slabs, max_batch=batch, **kw)
    return o, g


# every new node's one candidate is the one node there
@pytest.mark.parametrize("m", [3, 4, 5, 63, 64, 65, 128, 129, 256, 257, 512, 513, 577, 4095, 4096, 4097, 8192, 9000])
def test_one_hub(m):
    rng = np.random.default_rng(m)
    o, g = _pair(m + 40, m + 1, refine=False)
    for n in (1, m):
        x = rng.integers(0, 256, (n, DIM), dtype=np.uint8)
        o.insert(x)
        g.insert(_up(x))
    assert_same_state(o, g, "offered")
    gone = rng.permutation(np.arange(1, m + 1))[:max(1, m - 2)].astype(np.uint32)  # most of them, in no order
    so, sg = o.delete(gone), g.delete(_up(gone.view(np.int32)))
    assert np.array_equal(so, sg.cpu().numpy())
    assert_same_state(o, g, "repaired")
    g.close()


# a dozen hubs of very different degree in one launch, among nodes with a few pairs each
def test_hubs_of_many_sizes():
    rng = np.random.default_rng(7)
    centers = rng.integers(20, 236, (12, DIM)).astype(np.float64)
    sizes = [1, 2, 5, 30, 64, 70, 130, 300, 520, 700, 1500, 5000]
    label = rng.permutation(np.repeat(np.arange(12), sizes))
    o, g = _pair(12_000, label.size)
    rows = lambda c: np.clip(np.rint(centers[c] + 4 * rng.standard_normal((len(c), DIM))), 0, 255).astype(np.uint8)  # noqa: E731
    for c in (np.arange(12), label, rng.permutation(label)[:2000]):
        x = rows(c)
        o.insert(x)
        g.insert(_up(x))
        assert_same_state(o, g, f"{len(c)} inserted")
    gone = rng.permutation(np.arange(12, 12 + label.size + 2000))[:5000].astype(np.uint32)
    assert np.array_equal(o.delete(gone), g.delete(_up(gone.view(np.int32))).cpu().numpy())
    assert_same_state(o, g, "repaired")
    g.close()


def test_a_hubs_offers_cost_in_proportion():
    import torch
    from paper_2607_02543_amd import etale

    def us(m):
        best = 1e9
        for _ in range(3):
            g = etale.Index(DIM, R=R, L_build=12, n_entry=12, id_capacity=m + 8, slab_capacity=12 * m, max_batch=m, refine=False)
            x = torch.randint(0, 256, (m + 1, DIM), dtype=torch.uint8, device="cuda")
            g.insert(x[:1])
            torch.cuda.synchronize()
            t = time.perf_counter()
            g.insert(x[1:])
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
            g.close()
        return best * 1e6

    few, many = us(4096), us(16_384)
    print(f"[hub] 4,096 offers {few:.0f} us, 16,384 {many:.0f} us", flush=True)
    assert many < 6 * few  # n log^2 n; ranking every pair against every other is past ten times
