"""GPU tests of the ordered lookups' way back: answers written four at a time where the caller's
arrays are aligned for it and one at a time where they are not, at needle counts whose last tile
ends inside a group of four, with either output left out, and nothing written outside them."""
import pytest

from paper_2508_11443_amd import fks, workloads
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

M = 1 << 23
MISSING = 0x1234567


def _inputs(n, m):
    import torch
    keys = workloads.mix_keys_torch(torch.arange(n, device="cuda"))
    g = torch.Generator(device="cuda")
    g.manual_seed(m)
    at = torch.randint(0, 2 * n, (m,), generator=g, device="cuda")
    return keys, at, workloads.mix_keys_torch(at)


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("m,dv,df", [(M, 0, 0), (M + 1, 0, 1), (M + 2, 1, 0), (M + 3, 2, 3), (M + 61, 3, 2), (M + 64, 1, 1)])
def test_any_alignment_and_rest(m, dv, df, wide):
    import torch
    announce(f"gpu order return: m={m} offsets {dv} {df} wide={wide}")
    n = 1 << 20
    keys, at, q = _inputs(n, m)
    dt = torch.int64 if wide else torch.int32
    vals = torch.arange(n, dtype=dt, device="cuda") * 5 + 2
    want_f = (at < n).to(torch.uint8)
    want_v = torch.where(at < n, vals[at.clamp(max=n - 1)], torch.tensor(MISSING, dtype=dt, device="cuda"))
    build, lookup = (fks.fks_build_u64_v64, fks.fks_lookup_u64_v64) if wide else (fks.fks_build_u64, fks.fks_lookup_u64)
    mp = build(keys, vals, 3)
    for with_v, with_f in ((True, True), (True, False), (False, True)):
        if wide and not with_v:
            continue
        v = torch.full((m + 8,), -7, dtype=dt, device="cuda")
        f = torch.full((m + 8,), 9, dtype=torch.uint8, device="cuda")
        lookup(mp, q, v[dv:dv + m] if with_v else None, f[df:df + m] if with_f else None, MISSING)
        for out, want, d, given, guard in ((v, want_v, dv, with_v, -7), (f, want_f, df, with_f, 9)):
            if given:
                assert torch.equal(out[d:d + m], want)
                assert bool((out[:d] == guard).all()) and bool((out[d + m:] == guard).all())
            else:
                assert bool((out == guard).all())
    mp.destroy()
