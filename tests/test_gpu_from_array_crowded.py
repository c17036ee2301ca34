"""GPU test of from_array where keys crowd a pair of partitions under the partition hashes tried, with
more distinct keys than the pair's table in LDS has slots: the table equals the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2508_11443_amd import fks
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu

MASK = (1 << 64) - 1


def _bucket(x, sigma, r, n):
    a0, a1, b, _ = oracle.level1_consts(sigma, r)
    with np.errstate(over="ignore"):
        h = (np.uint64(a0) * (x & np.uint64(0xFFFFFFFF)) + np.uint64(a1) * (x >> np.uint64(32)) + np.uint64(b)) >> \
            np.uint64(32)
    return (h % np.uint64(n)).astype(np.int64)


def _crowded(distinct, crowd, u, seed, hashes):
    """u records of `distinct` keys, `crowd` of which lie in the first two partitions of 1024 buckets
    under each of the first `hashes` partition hashes (the level-one functions of seed ~seed)."""
    rng = np.random.default_rng(seed)
    got, count = [], 0
    while count < crowd:
        x = rng.integers(0, 2**64, size=1 << 20, dtype=np.uint64)
        for r in range(hashes):
            x = x[_bucket(x, ~seed & MASK, r, u) < 2048]
        got.append(x)
        count += x.size
    keys = np.unique(np.concatenate(got))[:crowd]
    keys = np.unique(np.concatenate([keys, rng.integers(0, 2**64, size=distinct - crowd, dtype=np.uint64),
                                     np.array([MASK], np.uint64)]))
    recs = np.concatenate([keys, keys[rng.integers(0, keys.size, size=u - keys.size)]])
    return rng.permutation(recs), rng.integers(0, 2**32, size=u, dtype=np.uint64).astype(np.uint32)


@pytest.mark.parametrize("u,distinct,crowd,hashes", [(16384, 14000, 6000, 1), (16384, 14000, 6000, 2),
                                                      (16384, 14000, 4200, 2), (300007, 40000, 9000, 2)])
def test_more_keys_than_a_pairs_table(u, distinct, crowd, hashes):
    seed = 0xC0D + u + hashes
    announce(f"gpu from_array crowded: u={u}, {crowd} keys in a pair under {hashes} hashes")
    keys, vals = _crowded(distinct, crowd, u, seed, hashes)
    assert crowd > 4096
    dk, dv = to_dev(keys), to_dev(vals)
    fks.fks_prof_reset()
    fks.fks_prof_enable(True)
    try:
        m = fks.fks_build_u64_from_array(dk, dv, seed)
        ran = fks.fks_prof_read()
    finally:
        fks.fks_prof_enable(False)
    assert ("fks_dedup_compact" in ran) == (hashes == 2)     # the table in device memory
    assert m.info()["n"] == np.unique(keys).size
    h, s, _ = fks.fks_export(m)
    rh, rs = oracle.build_u64_dedup(keys, vals, seed).export()
    assert (h == rh).all() and (s == rs).all()
    m.destroy()
