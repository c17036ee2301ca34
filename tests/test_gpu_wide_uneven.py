"""GPU test of a batch's large maps over keys that fall unevenly into partitions (consecutive integers,
multiples of a power of two, and such maps beside ones of spread keys): tables equal single builds', and such a batch takes at
most three times as long as one of spread keys (it took nine times as long where a workgroup gathered its
buckets' keys one by one)."""
import time

import numpy as np
import pytest

import oracle
from paper_2508_11443_amd import fks, workloads
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu


def _keys(kind, sizes, seed):
    total = int(sum(sizes))
    spread = workloads.unique_u64(total, seed, dense_fraction=0.0)
    run = np.arange(total, dtype=np.uint64)
    if kind == "multiples":
        return run << np.uint64(20)
    if kind == "consecutive":
        return run
    owner = np.repeat(np.arange(len(sizes)), sizes)
    return np.where(owner % 2 == 0, run, spread | np.uint64(1 << 63))


@pytest.mark.parametrize("kind", ["consecutive", "multiples", "every other map"])
def test_tables_equal_single_builds(kind):
    announce(f"gpu wide uneven: {kind}")
    sizes = [4096, 4097, 5121, 8192, 300, 30000, 65536, 20000, 4096, 16385, 50001, 65535]
    off = np.zeros(len(sizes) + 1, np.uint64)
    np.cumsum(np.array(sizes, np.uint64), out=off[1:])
    keys = _keys(kind, sizes, 9)
    vals = np.arange(keys.size, dtype=np.uint32)
    b = fks.fks_build_batch_u64(to_dev(keys), to_dev(vals), off, 77)
    for m in range(len(sizes)):
        lo, hi = int(off[m]), int(off[m + 1])
        h, s = fks.fks_batch_export(b, m)[:2]
        ref = oracle.build_u64(keys[lo:hi], vals[lo:hi], oracle.batch_seed(77, m))
        rh, rs = ref.export()
        assert (h == rh).all() and (s == rs).all(), (m, sizes[m])
    b.destroy()


def test_uneven_keys_take_no_longer():
    import torch
    M, n = 1000, 4096
    announce("gpu wide uneven: time")
    off = np.arange(M + 1, dtype=np.uint64) * np.uint64(n)
    vals = torch.arange(M * n, dtype=torch.int32, device="cuda")
    best = []
    for keys in (workloads.mix_keys_torch(torch.arange(M * n, device="cuda")), torch.arange(M * n, device="cuda")):
        times = []
        for _ in range(6):
            torch.cuda.synchronize()
            began = time.perf_counter()
            b = fks.fks_build_batch_u64(keys, vals, off, 5)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - began)
            b.destroy()
        best.append(min(times))
    assert best[1] < 3 * best[0], best
