"""GPU test of the partition passes at the sizes where their tiles change (2^18, 2^21 and 256 * 12288
keys) and at ragged tile ends, through the constructors that use them."""
import pytest

from paper_2508_11443_amd import fks, workloads
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1025, 2048, 2049, 6143, (1 << 18) - 1, 1 << 18, (1 << 18) + 1, (1 << 21) - 1, 1 << 21,
                               256 * 12288, 256 * 12288 + 1])
def test_every_key_is_found(n):
    import torch
    announce(f"gpu tiles: n={n}")
    keys = workloads.mix_keys_torch(torch.arange(n, device="cuda"))
    vals = torch.arange(n, dtype=torch.int32, device="cuda")
    wide = workloads.mix_keys_torch(torch.arange(n, 2 * n, device="cuda"))
    v = torch.empty(n, dtype=torch.int32, device="cuda")
    w = torch.empty(n, dtype=torch.int64, device="cuda")
    f = torch.empty(n, dtype=torch.uint8, device="cuda")
    m = fks.fks_build_u64(keys, vals, n)
    fks.fks_lookup_u64(m, keys, v, f)
    assert bool(f.all()) and torch.equal(v, vals)
    m.destroy()
    m = fks.fks_build_u64_v64(keys, wide, n)
    fks.fks_lookup_u64_v64(m, keys, w, f)
    assert bool(f.all()) and torch.equal(w, wide)
    m.destroy()
    m = fks.fks_build_u64_from_array(torch.cat([keys, keys]), torch.cat([vals, vals + 7]), n)
    assert m.info()["n"] == n
    fks.fks_lookup_u64(m, keys, v, f)
    assert bool(f.all()) and torch.equal(v, vals)
    m.destroy()
