"""Start-set scoring: with every row in the entry set, a query's initial list
holds its exact nearest rows, so a search returns them whatever the graph.
Compared with the plain definition, by (distance, id), at the edges of the
groups (4 and 32 rows), spans (256), selection steps (4,096), list lengths and
of the rules that choose between the written matrix and the bounded keys, with
rows of a few distinct values (more ties at the bound than the key list takes)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def nearest(x, q, live, k, u8):
    if u8:
        a, b = q.astype(np.int64), x[live].astype(np.int64)
        d = (a * a).sum(1)[:, None] + (b * b).sum(1)[None, :] - 2 * (a @ b.T)
    else:
        d = 1.0 - q.astype(np.float64) @ x[live].T.astype(np.float64)
    order = np.argsort(d, axis=1, kind="stable")[:, :k]  # live ids ascend
    return live[order], np.take_along_axis(d, order, 1)


def build(x, u8):
    import torch

    from paper_2607_02543_amd import etale
    n, dim = x.shape
    g = etale.Index(dim, R=8, L_build=16, n_entry=n, id_capacity=n + 8, max_batch=n, W=2,
                    metric=etale.METRIC_L2_U8 if u8 else etale.METRIC_IP_F32)
    g.insert(torch.from_numpy(x).cuda())
    return g


def check(g, x, q, live, Ls, u8):
    import torch
    qd = torch.from_numpy(q).cuda()
    for L in Ls:
        k = min(10, L)
        ids, d = nearest(x, q, live, k, u8)
        gi, gd = g.search(qd, k, L)
        assert np.array_equal(ids, gi.cpu().numpy()[:, :ids.shape[1]])
        assert np.array_equal(d, gd.cpu().numpy()[:, :ids.shape[1]].astype(d.dtype))


@pytest.mark.parametrize("dim", [64, 128, 256])
@pytest.mark.parametrize("n,nq,values", [
    (31, 1, 256), (257, 65, 256), (1001, 33, 256), (2048, 64, 256), (4096, 5, 256), (4099, 7, 256),
    (4099, 2100, 256),  # past the matrix rule for lists below n / 32
    (3000, 9, 2), (6002, 3, 2),  # few distinct rows: thousands of ties
])
def test_uint8_start_lists(dim, n, nq, values):
    import torch
    rng = np.random.default_rng(dim + n)
    if values == 2:
        x = rng.integers(0, 256, (3, dim), dtype=np.uint8)[rng.integers(0, 3, n)]
    else:
        x = rng.integers(0, 256, (n, dim), dtype=np.uint8)
    q = rng.integers(0, 256, (nq, dim), dtype=np.uint8)
    g = build(x, True)
    check(g, x, q, np.arange(n), (16, 64, 128), True)
    gone = np.arange(0, n, 5)
    g.delete(torch.from_numpy(gone.astype(np.int32)).cuda())
    check(g, x, q, np.setdiff1d(np.arange(n), gone), (16, 64, 128), True)
    g.close()


# values in eighths with few of them nonzero: every order of summation is exact
@pytest.mark.parametrize("dim,n,nq", [(96, 33, 1), (96, 1001, 130), (96, 4099, 2100), (192, 257, 17), (384, 700, 600),
                                      (768, 300, 33)])
def test_float_start_lists(dim, n, nq):
    rng = np.random.default_rng(dim + n)
    x = (rng.integers(-2, 3, (n, dim)) / 8).astype(np.float32)
    q = (rng.integers(-2, 3, (nq, dim)) / 8).astype(np.float32)
    g = build(x, False)
    check(g, x, q, np.arange(n), (16, 64, 128), False)
    g.close()
