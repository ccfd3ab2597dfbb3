"""The device-wide heap engine at the edges of its steps: tiles of 2048, groups
of 64 tiles, the compaction's tiles, Select with no, one and several passes
(even, crowded and equal keys), and the two sorts of the extracted minima."""
import numpy as np
import pytest
import torch

import oracle
import paper_1908_09378_amd as pkg
from gpu_util import DEV, dev32, dev64, host32, host64

pytestmark = pytest.mark.gpu


def keys_of(rng, kind, n):
    if kind == "even":
        return rng.integers(0, 1 << 40, n, dtype=np.uint64)
    if kind == "crowded":  # half of them in the lowest 2^-20 of the range
        k = rng.integers(0, 1 << 40, n, dtype=np.uint64)
        return np.where(rng.random(n) < 0.5, k >> np.uint64(20), k).astype(np.uint64)
    if kind == "two":
        return np.where(rng.random(n) < 0.5, np.uint64(5), np.uint64((1 << 64) - 2))
    return np.full(n, 77, np.uint64)


def run(cap, d, kind, batches, takes, deletes, seed):
    rng = np.random.default_rng(seed)
    h, o = pkg.Heap(cap, d, pkg.ENGINE_WIDE, 0), oracle.PQ(cap)
    for r, n in enumerate(batches):
        ids = rng.permutation(cap)[:n].astype(np.uint32)
        keys = keys_of(rng, kind, n)
        h.bulk_update(dev64(keys), dev32(ids))
        o.bulk_update(keys, ids)
        if deletes:
            gone = rng.integers(0, cap, deletes).astype(np.uint32)
            h.delete(dev32(gone))
            o.delete(gone)
        t = takes[r % len(takes)]
        ok, oi = torch.zeros(t, dtype=torch.int64, device=DEV), torch.zeros(t, dtype=torch.int32, device=DEV)
        got = h.extract_min(t, ok, oi)
        wk, wi = o.extract_min(t)
        assert got == len(wk)
        assert np.array_equal(host64(ok)[:got], wk) and np.array_equal(host32(oi)[:got], wi)
        assert h.size() == o.size()


@pytest.mark.parametrize("kind", ["even", "crowded", "two", "equal"])
@pytest.mark.parametrize("d", [2047, 2048, 4099, 9000, 65536])
def test_steps(kind, d):
    cap = 3 * d + 17
    run(cap, d, kind, [cap, d, 1, d - 1, 2 * d + 1, cap], [d // 2, 3, d, 2 * d], 0, d)


@pytest.mark.parametrize("take", [1, 31, 33, 4095, 4096, 4097, 12287, 12288, 12289, 16384, 16385, 40000])
def test_extract_sorts(take):
    run(120000, 30000, "even", [120000, 30000, 5000], [take], 900, take)


@pytest.mark.parametrize("cap", [31, 512 * 32, 512 * 32 + 1, 64 * 512 * 32 + 3])
def test_compaction_tiles(cap):
    run(cap, min(cap, 20000), "even", [cap, max(1, cap // 3)], [min(cap, 5000)], 0, cap)


def test_growth_between_steps():
    """More elements than the first levels hold: the arena and the scratch grow
    while B_0 keeps its key range."""
    run(1 << 20, 1024, "crowded", [1 << 16, 1 << 18, 1 << 20, 5, 1 << 19], [2000, 1, 70000], 100, 9)


@pytest.mark.parametrize("engine", [pkg.ENGINE_TEAM, pkg.ENGINE_WIDE])
@pytest.mark.parametrize("n", [1, 511, 513, 131072, 524289])
def test_batch_check(engine, n):
    """One bad pair anywhere in a batch refuses it whole, and the next call is
    judged by its own batch."""
    h = pkg.Heap(n, 4096, engine)
    keys, ids = np.arange(n, dtype=np.uint64), np.arange(n, dtype=np.uint32)
    for at in sorted({0, n // 2, n - 1}):
        bad = ids.copy()
        bad[at] = n
        low = keys.copy()
        low[at] = (1 << 64) - 1
        for call in (lambda: h.bulk_update(dev64(keys), dev32(bad)), lambda: h.bulk_update(dev64(low), dev32(ids)),
                     lambda: h.delete(dev32(bad))):
            with pytest.raises(pkg.PBHError) as e:
                call()
            assert e.value.code == pkg.PBH_EINVAL
        h.delete(dev32(ids))
        assert h.size() == 0
    h.bulk_update(dev64(keys), dev32(ids))
    assert h.size() == n
