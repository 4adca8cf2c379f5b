"""Reclaim's two passes against the exported lists: the dirty nodes and dead
edges it counts are those of the state before it, and each list afterwards is
the list before it without its deleted entries, in order. Lists in whole
16-byte words (R = 8, 48) and not (R = 6), fewer and more ids than the bits of
the workgroups' own bitmap (2^20), one and several batches of nodes per wave."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R", [(70, 6), (1500, 48), (1025, 8), (40_000, 6), ((1 << 20) + 3000, 8)])
def test_reclaim_lists(n, R):
    import torch

    from paper_2607_02543_amd import etale
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + R)
    x = torch.randint(0, 256, (n, 64), dtype=torch.uint8, device="cuda", generator=gen)
    batch = min(n, 16_000)
    g = etale.Index(64, R=R, L_build=16, n_entry=64, id_capacity=n + 8, max_batch=batch, refine=False,
                    slab_capacity=2 * n + 3 * batch * (R + 2))
    done, b = 0, min(n, 1000)
    while done < n:
        g.insert(x[done:done + b])
        done += b
        b = min(batch, max(done, 1), n - done)
    gone = torch.randperm(n, device="cuda", generator=gen)[:max(7, min(n // 5, batch))].to(torch.int32)
    g.delete(gone)
    a = g.export()
    g.reclaim()
    s, z = g.stats(), g.export()
    live = ~a["deleted"]
    used = np.arange(R)[None, :] < a["deg"][:, None]
    dead = used & a["deleted"][np.where(used, a["nbr"], 0)] & live[:, None]
    assert dead.any()
    assert s["dirty_last"] == int(dead.any(1).sum()) and s["dead_edges_last"] == int(dead.sum())
    keep = used & ~dead & live[:, None]
    assert np.array_equal(z["deg"][live], keep.sum(1)[live])
    left = np.arange(R)[None, :] < z["deg"][:, None]
    left &= live[:, None]
    assert np.array_equal(z["nbr"][left], a["nbr"][keep]) and np.array_equal(z["rho"][left], a["rho"][keep])
    assert not z["has_slab"][~live].any()
    g.close()
