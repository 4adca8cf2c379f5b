"""The float brute force where its passes meet their limits: every distance tied, and more queries than one pass of
group minima holds."""

import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _index(n, dim, seed, max_batch=16_384):
    import torch
    from paper_2607_02543_amd import etale
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    x = torch.randn((n, dim), device="cuda", generator=gen)
    x /= x.norm(dim=1, keepdim=True)
    g = etale.Index(dim, R=4, L_build=8, n_entry=16, id_capacity=n, slab_capacity=2 * n + 8 * max_batch,
                    max_batch=max_batch, refine=False, metric=etale.METRIC_IP_F32)
    for b in range(0, n, max_batch):
        g.insert(x[b:b + max_batch])
    return g, x, gen


# a zero query is at distance 1 from every row: every group is at the bound
def test_tied_distances_cost_what_others_do():
    import torch
    g, _, gen = _index(65_536, 96, 1)
    q = torch.randn((500, 96), device="cuda", generator=gen)
    z = torch.zeros_like(q)

    def us(q):
        best = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            g.bruteforce(q, 10)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best * 1e6

    other, tied = us(q), us(z)
    print(f"[bruteforce] {other:.0f} us, tied {tied:.0f} us", flush=True)
    assert tied < 2 * other + 200  # rescoring every group takes ten times as long
    gone = np.arange(0, 40, 3)
    g.delete(torch.from_numpy(gone.astype(np.int32)).cuda())
    i, d = g.bruteforce(z, 16)
    want = np.setdiff1d(np.arange(40), gone)[:16]
    assert np.array_equal(i.cpu().numpy(), np.tile(want, (500, 1))) and bool((d == 1.0).all())
    g.close()


def _same(a, b):
    import torch
    return torch.equal(a[0], b[0]) and torch.equal(a[1].view(torch.int32), b[1].view(torch.int32))


# a wave takes 32 queries (16 from 384 dimensions on): batches that end before, at and past a block
@pytest.mark.parametrize("dim", [96, 192, 384, 768])
def test_a_batch_gives_what_its_queries_give_alone(dim):
    import torch
    g, _, gen = _index(700, dim, dim, max_batch=350)
    q = torch.randn((33, dim), device="cuda", generator=gen)
    alone = [g.bruteforce(q[i:i + 1], 16) for i in range(33)]
    for n in (15, 16, 17, 31, 32, 33):
        i, d = g.bruteforce(q[:n], 16)
        assert _same((i, d), (torch.cat([a[0] for a in alone[:n]]), torch.cat([a[1] for a in alone[:n]]))), n
    g.close()


# the group minima of 65,536 rows fill their 256 MiB at 65,536 queries; one group's launch ends at 2^23 queries
@pytest.mark.parametrize("n,split", [(65_536, 65_536), (64, 1 << 23)])
def test_more_queries_than_one_launch_holds(n, split):
    import torch
    g, _, gen = _index(n, 96, n, max_batch=min(n, 16_384))
    q = torch.randn((split + 33, 96), device="cuda", generator=gen)
    i, d = g.bruteforce(q, 5)
    for b, e in ((0, 40), (split - 40, split), (split - 1, split + 1), (split, split + 33)):
        assert _same((i[b:e].contiguous(), d[b:e].contiguous()), g.bruteforce(q[b:e].contiguous(), 5)), (b, e)
    g.close()
