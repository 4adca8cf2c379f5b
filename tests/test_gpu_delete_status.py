"""Statuses of delete batches whose ids repeat, lie past the ids handed out or past the id space, and their cost."""

import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CAP, BORN = 5000, 1200


def _index(max_batch, cap=CAP):
    import torch
    from paper_2607_02543_amd import etale
    g = etale.Index(16, R=4, L_build=8, n_entry=16, id_capacity=cap, slab_capacity=4 * cap + 6 * max_batch,
                    max_batch=max_batch)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    x = torch.randint(0, 256, (BORN, 16), dtype=torch.uint8, device="cuda", generator=gen)
    for b in range(0, BORN, 600):
        g.insert(x[b:b + 600])
    return g


# batches of one and several workgroups; ids that share their low bits (and with them their place in a hash table), the
# last ids of 32 bits, many repeats of few ids
@pytest.mark.parametrize("n,kind", [(1, "far"), (63, "far"), (700, "mixed"), (700, "one"), (2500, "mixed"), (2500, "low"),
                                    (2500, "far"), (2500, "few")])
def test_statuses(n, kind):
    import torch
    rng = np.random.default_rng(n)
    g = _index(2500)
    gone = np.zeros(BORN, bool)
    for _ in range(4):
        far = np.concatenate([rng.integers(CAP, 1 << 32, n), (np.arange(n) << 14) + CAP, (1 << 32) - 1 - np.arange(n)])
        ids = {"far": rng.choice(far, n), "low": rng.choice((np.arange(1 << 17) << 13) + 9, n),
               "few": rng.choice([3, 4000, CAP, CAP + 1, 1 << 20, (1 << 32) - 1], n), "one": np.full(n, CAP + 7),
               "mixed": rng.choice(np.concatenate([np.arange(0, CAP, 3), rng.choice(far, 800)]), n)}[kind].astype(np.uint32)
        want = np.zeros(n, np.uint8)
        seen = set()
        for t, i in enumerate(ids.tolist()):
            want[t] = 3 if i in seen else 2 if i >= BORN else 1 if gone[i] else 0
            seen.add(i)
            if i < BORN:
                gone[i] = True
        got = g.delete(torch.from_numpy(ids.view(np.int32)).cuda()).cpu().numpy()
        assert np.array_equal(got, want)
    st = g.stats()
    assert st["live"] == BORN - int(gone.sum()) and st["error_bits"] == 0
    g.close()


def test_ids_never_handed_out_cost_what_others_do():
    import torch
    n = 131_072
    g = _index(n, cap=2 * n)
    sync = torch.cuda.synchronize

    def us(ids):
        best = 1e9
        for _ in range(5):
            sync()
            t = time.perf_counter()
            g.delete(ids)
            sync()
            best = min(best, time.perf_counter() - t)
        return best * 1e6

    at = torch.arange(n, device="cuda", dtype=torch.int32)
    g.delete(at[:BORN // 2].clone())
    known = us((at % (BORN // 2)))  # deleted already
    for ids in (at + BORN, at + 3 * n):
        cost = us(ids)
        print(f"[delete] {n} ids: {known:.0f} us handed out, {cost:.0f} us not", flush=True)
        assert cost < 5 * known + 500  # a search of the earlier positions for each takes fifty times as long
    g.close()
