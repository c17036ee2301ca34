"""GPU test of many needles against comparison maps of few keys, on both sides of the sizes where each
lane searches alone: every key, its neighbours and the extremes, with and without values, against
numpy's binary search; and the time of such a search, which grows with the number of keys."""
import numpy as np
import pytest

from paper_2508_11443_amd import fks, workloads
from tests.gpu_util import announce, empty, to_dev, to_np

pytestmark = pytest.mark.gpu

MISSING = 0xFFFFFFFE
ONES = np.uint64(2**64 - 1)


@pytest.mark.parametrize("layout,n", [(0, 1), (0, 2), (0, 3), (0, 255), (0, 256), (0, 257), (1, 1), (1, 2), (1, 3), (1, 4),
                                      (1, 4095), (1, 4096), (1, 4097), (1, 16383), (1, 16384), (1, 16385)])
def test_every_key_and_its_neighbours(layout, n):
    announce(f"gpu small search: layout={layout} n={n}")
    rng = np.random.default_rng(n)
    keys = workloads.unique_u64(n, n + layout, dense_fraction=0.5)
    if n > 3:
        keys[:2] = 0, ONES
    keys = rng.permutation(np.unique(keys))
    vals = rng.integers(0, 2**32, size=keys.size, dtype=np.uint64).astype(np.uint32)
    s = fks.fks_sorted_build_u64(to_dev(keys), to_dev(vals), layout)
    order = np.argsort(keys)
    near = np.concatenate([keys, keys + np.uint64(1), keys - np.uint64(1), np.array([0, 1, ONES], np.uint64)])
    for m in ((1 << 19) - 1, 1 << 19, (1 << 20) - 1, 1 << 20, (1 << 20) + 1021):
        q = near[rng.integers(0, near.size, size=m)]
        q[:min(m, near.size)] = near[:m]
        at = np.minimum(np.searchsorted(keys[order], q), keys.size - 1)
        hit = keys[order][at] == q
        v, f = empty(m, "u32"), empty(m, "u8")
        fks.fks_sorted_lookup_u64(s, to_dev(q), v, f, missing=MISSING)
        assert (to_np(f, "u8") == hit).all()
        assert (to_np(v, "u32") == np.where(hit, vals[order][at], np.uint32(MISSING))).all()
        f.fill_(7)
        fks.fks_sorted_lookup_u64(s, to_dev(q), None, f, missing=MISSING)
        assert (to_np(f, "u8") == hit).all()
    s.destroy()


@pytest.mark.parametrize("layout", [0, 1])
def test_few_keys_take_less_time_than_many(layout):
    """16 keys against 2^20: at least three times faster (needles in, answers out: the floor is 20 us)."""
    import torch
    m = 1 << 23
    announce(f"gpu small search: time, layout={layout}")
    times = []
    for n in (16, 1 << 20):
        keys = workloads.mix_keys_torch(torch.arange(n, device="cuda"))
        s = fks.fks_sorted_build_u64(keys, torch.arange(n, dtype=torch.int32, device="cuda"), layout)
        q = keys[torch.randint(0, n, (m,), device="cuda")]
        v, f = empty(m, "u32"), empty(m, "u8")
        best = 1e9
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            fks.fks_sorted_lookup_u64(s, q, v, f)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
        s.destroy()
    assert 3 * times[0] < times[1], times
