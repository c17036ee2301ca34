"""GPU test of a batch's maps at the sizes where the partition passes take them over (4096 keys)
and where their tiles (4096 records) and partitions (1024 buckets) begin, beside small and
empty maps, against single builds with the maps' seeds."""
import numpy as np
import pytest

import oracle
from paper_2508_11443_amd import workloads
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu

SIZES = [4095, 4096, 4097, 0, 5120, 5121, 8191, 8192, 8193, 1, 12289, 65535, 65536, 300, 16385, 4096]


@pytest.mark.parametrize("order", ["given", "reversed"])
def test_tables_equal_single_builds(order):
    from paper_2508_11443_amd import fks
    announce(f"gpu wide maps: {order}")
    sizes = SIZES if order == "given" else SIZES[::-1]
    off = np.zeros(len(sizes) + 1, np.uint64)
    np.cumsum(np.array(sizes, np.uint64), out=off[1:])
    keys = workloads.unique_u64(int(off[-1]), 77, dense_fraction=0.4)
    vals = np.arange(keys.size, dtype=np.uint32)
    b = fks.fks_build_batch_u64(to_dev(keys), to_dev(vals), off, 4242)
    for m, n in enumerate(sizes):
        lo, hi = int(off[m]), int(off[m + 1])
        h, s = fks.fks_batch_export(b, m)[:2]
        ref = oracle.build_u64(keys[lo:hi], vals[lo:hi], oracle.batch_seed(4242, m)) if n else None
        if n:
            rh, rs = ref.export()
            assert (h == rh).all() and (s == rs).all(), (m, n)
    b.destroy()
