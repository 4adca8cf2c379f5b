"""Visited-table slots: a count that a caller sets is the one that runs, whatever the launch's size, and the default never
costs more than a count that could be set."""

import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _index(dim, n, seed, **kw):
    import torch
    from paper_2607_02543_amd import etale
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    u8 = kw.get("metric", etale.METRIC_L2_U8) == etale.METRIC_L2_U8
    if u8:
        make = lambda m: torch.randint(0, 256, (m, dim), dtype=torch.uint8, device="cuda", generator=gen)  # noqa: E731
    else:
        def make(m):
            c = torch.randn((500, dim), device="cuda", generator=torch.Generator(device="cuda").manual_seed(9))
            x = c[torch.randint(0, 500, (m,), device="cuda", generator=gen)] / dim ** 0.5
            x = x + 0.3 * torch.randn((m, dim), device="cuda", generator=gen)
            return x / x.norm(dim=1, keepdim=True)
    g = etale.Index(dim, id_capacity=n, slab_capacity=3 * n + 70_000, max_batch=2000, **kw)
    x = make(n)
    for b in range(0, n, 2000):
        g.insert(x[b:b + 2000])
    return g, make


# few queries, whose launch has room for any table: a table too small for a search repeats distances
@pytest.mark.parametrize("metric,dim,W,L", [(0, 128, 1, 64), (0, 128, 2, 101), (0, 64, 4, 32), (1, 96, 1, 64), (1, 96, 2, 100)])
def test_a_set_count_is_the_one_that_runs(metric, dim, W, L):
    import torch
    kw = dict(R=32, L_build=64, n_entry=64, W=W, metric=metric)
    scored = {}
    for at_create in (True, False):
        for slots in (64, 4096):
            g, make = _index(dim, 4000, 5, vt_slots=slots if at_create else 1024, **kw)
            if not at_create:
                g.set_search_knobs(4, slots)
            q = make(200)
            i, d, c = g.search(q, 10, L, counts=True)
            scored[at_create, slots] = (int(c[:, 1].sum()), i, d)
            g.close()
    for at_create in (True, False):
        few, many = scored[at_create, 64], scored[at_create, 4096]
        assert torch.equal(few[1], many[1]) and torch.equal(few[2], many[2])
        assert few[0] > 1.2 * many[0], (few[0], many[0])
    assert scored[True, 64][0] == scored[False, 64][0] and scored[True, 4096][0] == scored[False, 4096][0]


# lists in LDS: where that bounds the resident waves a large table costs more than it saves, unless a distance is dear
@pytest.mark.parametrize("dim,trav,W,L", [(96, 0, 1, 160), (96, 0, 4, 100), (768, 0, 1, 160), (384, 2, 1, 160)])
def test_the_default_is_no_slower_than_a_set_count(dim, trav, W, L):
    import torch
    n = 30_000 if dim == 96 else 8000
    g, make = _index(dim, n, 6, R=16 if dim == 96 else 32, L_build=48, n_entry=1024, W=W, metric=1, traversal=trav)
    q = make(3000)

    def us():
        best = 1e9
        for _ in range(8):
            torch.cuda.synchronize()
            t = time.perf_counter()
            g.search(q, 10, L)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best * 1e6

    default, found = us(), g.search(q, 10, L)
    others = {}
    for slots in (512, 2048, 4096):
        g.set_search_knobs(4, slots)
        others[slots] = us()
        assert all(torch.equal(a, b) for a, b in zip(found, g.search(q, 10, L)))
    print(f"[visited] {dim}-d {trav} W={W} L={L}: default {default:.0f} us, set {others}", flush=True)
    assert default < 1.15 * min(others.values())
    g.close()
