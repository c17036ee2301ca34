"""GPU tests of the comparison maps' separator search at the sizes where a line or a level of
separators begins or ends, with every key, its neighbours and the extreme words as needles."""
import numpy as np
import pytest

import oracle
from paper_2508_11443_amd import workloads
from tests.gpu_util import announce
from tests.test_gpu_search import MISSING, _fks, gpu_lookup
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("n", [15, 16, 17, 31, 32, 33, 255, 256, 257, 65535, 65536, 65537, 131071, 131072,
                               (1 << 20) - 1, 1 << 20, (1 << 20) + 17])
def test_every_key_and_its_neighbours(layout, n):
    announce(f"gpu separators: layout={layout} n={n}")
    keys = workloads.unique_u64(n, n + layout, dense_fraction=0.3)
    keys[0] = np.uint64(2**64 - 1) if not (keys == np.uint64(2**64 - 1)).any() else keys[0]
    vals = np.random.default_rng(n).integers(0, 2**32, size=n, dtype=np.uint32)
    s = _fks().fks_sorted_build_u64(to_dev(keys), to_dev(vals), layout)
    rk, rv = oracle.search_build(keys, vals, layout)
    q = np.concatenate([keys, keys + np.uint64(1), keys - np.uint64(1), np.array([0, 2**63, 2**64 - 1], np.uint64)])
    v, f = gpu_lookup(s, q)
    ov, of = oracle.search_lookup(rk, rv, layout, q, missing=MISSING)
    assert (f == of).all() and (v == ov).all()
