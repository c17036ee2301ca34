"""GPU test of the cells a build takes before it knows the table's size: keys whose table is far
above and far below the estimate, from the library's memory (the rest goes back) and from a
caller's allocator (the final pass runs again), give the oracle's bytes."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_single import skewed_keys
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3000, 40000, 300000])
@pytest.mark.parametrize("own", [True, False])
def test_table_far_above_the_estimate(n, own):
    from paper_2508_11443_amd import fks
    seed = 0xCE11 + n
    announce(f"gpu cells: n={n} own={own}")
    keys = skewed_keys(n, seed, 3, n)
    vals = np.arange(n, dtype=np.uint32)
    ref = oracle.build_u64(keys, vals, seed)
    assert ref.S > 2.5 * n
    maps = [fks.fks_build_u64(to_dev(keys), to_dev(vals), seed, allocator=None if own else fks.torch_allocator())
            for _ in range(3)]       # the returned ends are handed to the next map
    for m in maps:
        h, s, _ = fks.fks_export(m)
        rh, rs = ref.export()
        assert (h == rh).all() and (s == rs).all()
        if own:
            i = m.info()
            assert i["device_bytes"] == i["header_bytes"] + i["slot_bytes"] + 24 * i["T"]
        m.destroy()
