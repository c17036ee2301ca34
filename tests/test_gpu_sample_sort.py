"""GPU tests of the comparison maps' sample sort: sizes where a leaf, a bucket or a level of
splitters begins (3584 pairs in a leaf, 1344 on average, 256 leaves in a bucket), and keys that
are not spread evenly (sorted, reversed, dense runs, clusters of every magnitude)."""
import numpy as np
import pytest

from paper_2508_11443_amd import workloads
from tests import searchcheck
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3583, 3584, 3585, 1344 * 256, 1344 * 256 + 1, 2048 * 300 + 7, (1 << 21) + 5, 5242880 + 3]


def _fks():
    from paper_2508_11443_amd import fks
    return fks


def _clusters(n):
    """Distinct keys at every magnitude: runs of consecutive words around 2^(i/4)."""
    per = n // 200 + 1
    starts = (2.0 ** (20 + np.arange(200) * 0.21)).astype(np.uint64)
    keys = (starts[:, None] + np.arange(per, dtype=np.uint64)[None, :]).reshape(-1)
    return np.unique(keys)


def _keys(kind, n):
    rng = np.random.default_rng(n)
    if kind == "clusters":
        k = _clusters(4 * n)[:]
        return rng.permutation(k)[:n] if k.size >= n else workloads.unique_u64(n, n)
    k = workloads.unique_u64(n, n, dense_fraction={"even": 0.0, "half dense": 0.5}.get(kind, 0.1))
    if kind == "ascending":
        k = np.sort(k)
    if kind == "descending":
        k = np.sort(k)[::-1].copy()
    return k


@pytest.mark.parametrize("kind", ["even", "half dense", "ascending", "descending", "clusters"])
@pytest.mark.parametrize("n", SIZES)
def test_sorted_pairs(kind, n):
    fks = _fks()
    announce(f"gpu sample sort: {kind} n={n}")
    keys = _keys(kind, n)
    assert keys.size == n
    vals = np.random.default_rng(n + 1).integers(0, 2**32, size=n, dtype=np.uint32)
    order = np.argsort(keys)
    dk, dv = to_dev(keys), to_dev(vals)
    s = fks.fks_sorted_build_u64(dk, dv, 0)
    gk, gv = fks.fks_sorted_export(s)
    assert (gk == keys[order]).all() and (gv == vals[order]).all()
    e = fks.fks_sorted_build_u64(dk, dv, 1)
    gk, gv = fks.fks_sorted_export(e)
    nodes = np.unique(np.concatenate([np.arange(1, min(n, 40) + 1),
                                      np.random.default_rng(2).integers(1, n + 1, size=300), [n]]))
    for i in nodes.tolist():
        r = order[searchcheck.inorder_rank(i, n)]
        assert gk[i - 1] == keys[r] and gv[i - 1] == vals[r]
    assert (np.sort(gk) == keys[order]).all()


@pytest.mark.parametrize("n,repeats", [(3000, 2), (400000, 2), (400000, 400000), (3000000, 2000)])
def test_equal_keys_are_reported(n, repeats):
    """One repeated key, and so many of them that a leaf cannot hold them."""
    fks = _fks()
    announce(f"gpu sample sort: {repeats} equal keys of {n}")
    keys = workloads.unique_u64(n, 5)
    keys[np.random.default_rng(n).permutation(n)[:repeats]] = keys[0]
    for layout in (0, 1):
        with pytest.raises(fks.FksError) as err:
            fks.fks_sorted_build_u64(to_dev(keys), to_dev(np.zeros(n, np.uint32)), layout)
        assert err.value.code == fks.FKS_EDUPKEY


def test_same_layout_with_a_callers_allocator():
    """A caller's allocator keeps the radix sort: the two agree."""
    fks = _fks()
    announce("gpu sample sort: against the radix sort")
    n = 700001
    keys, vals = workloads.unique_u64(n, 9, dense_fraction=0.4), np.arange(n, dtype=np.uint32)
    for layout in (0, 1):
        a = fks.fks_sorted_export(fks.fks_sorted_build_u64(to_dev(keys), to_dev(vals), layout))
        b = fks.fks_sorted_export(fks.fks_sorted_build_u64(to_dev(keys), to_dev(vals), layout,
                                                           allocator=fks.torch_allocator()))
        assert (a[0] == b[0]).all() and (a[1] == b[1]).all()
