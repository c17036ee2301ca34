"""GPU tests of from_array's partitioned deduplication at the sizes where its plan changes (one
partition, the first pair, one scatter pass, two) and for repeats that crowd a partition: the
table equals the oracle's from_array byte for byte."""
import numpy as np
import pytest

import oracle
from paper_2508_11443_amd import fks, workloads
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu

ONES = np.uint64(2**64 - 1)


def _repeated(u, distinct, hot, seed):
    """u keys drawn from `distinct`; a share `hot` of them is one key (the all-ones key among
    the rest)."""
    rng = np.random.default_rng(seed)
    pool = workloads.unique_u64(distinct, seed + 1)
    if distinct > 1:
        pool[0] = ONES
    keys = pool[rng.integers(0, distinct, size=u)]
    keys[rng.random(u) < hot] = pool[distinct // 2]
    return keys, rng.integers(0, 2**32, size=u, dtype=np.uint64).astype(np.uint32)


@pytest.mark.parametrize("u,distinct,hot", [
    (2, 1, 0.0), (1024, 1 << 40, 0.0), (1025, 700, 0.0), (2049, 1 << 40, 0.0), (3073, 1, 0.0),
    ((1 << 18) - 1, 200000, 0.0), ((1 << 18) + 1, 1 << 40, 0.0), (300007, 100, 0.0),
    (300007, 150000, 0.5), ((1 << 20) + 77, 1 << 40, 0.01)])
def test_from_array_plan_edges(u, distinct, hot):
    distinct = min(distinct, u)
    announce(f"gpu from_array edges: u={u} distinct={distinct} hot={hot}")
    keys, vals = _repeated(u, distinct, hot, u)
    m = fks.fks_build_u64_from_array(to_dev(keys), to_dev(vals), 5 + u)
    ref = oracle.build_u64_dedup(keys, vals, 5 + u)
    assert m.info()["n"] == np.unique(keys).size
    h, s, _ = fks.fks_export(m)
    rh, rs = ref.export()
    assert (h == rh).all() and (s == rs).all()


def test_from_array_all_ones_only():
    announce("gpu from_array: the all-ones key alone, repeated")
    keys = np.full(5000, ONES, np.uint64)
    vals = np.arange(7, 5007).astype(np.uint32)
    m = fks.fks_build_u64_from_array(to_dev(keys), to_dev(vals), 3)
    h, s, _ = fks.fks_export(m)
    rh, rs = oracle.build_u64_dedup(keys, vals, 3).export()
    assert m.info()["n"] == 1 and (h == rh).all() and (s == rs).all()
