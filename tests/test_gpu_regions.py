"""GPU test of the partition passes at the sizes where every XCD gets regions of its own (2^24
records with an aux word, 2^25 without): every key is found with its value."""
import pytest

from paper_2508_11443_amd import fks, workloads
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n", [("u32", (1 << 25) - 1), ("u32", 1 << 25), ("u32", 40000003), ("u64", (1 << 24) - 1),
                                    ("u64", 1 << 24), ("u64", 20000003)])
def test_every_key_is_found(kind, n):
    import torch
    announce(f"gpu regions: {kind} n={n}")
    keys = workloads.mix_keys_torch(torch.arange(n, device="cuda"))
    f = torch.empty(n, dtype=torch.uint8, device="cuda")
    if kind == "u32":
        vals = torch.arange(n, dtype=torch.int32, device="cuda")
        v = torch.empty_like(vals)
        m = fks.fks_build_u64(keys, vals, n)
        fks.fks_lookup_u64(m, keys, v, f)
    else:
        vals = workloads.mix_keys_torch(torch.arange(n, 2 * n, device="cuda"))
        v = torch.empty_like(vals)
        m = fks.fks_build_u64_v64(keys, vals, n)
        fks.fks_lookup_u64_v64(m, keys, v, f)
    assert bool(f.all()) and torch.equal(v, vals)
    m.destroy()
