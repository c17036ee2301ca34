"""GPU tests of the ordered lookups (many needles against a large table): answers against the way
the needles were made, at the smallest sizes that take the path, at ragged tile ends and beyond
one slice, for needles that all fall into one part, on side streams one call behind the other,
with and without either output, and against the direct path under graph capture."""
import numpy as np
import pytest

from paper_2508_11443_amd import fks, workloads
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

MISSING = 0xABCDEF01
TILE, TILE_IDS = 15360, 12288


def _table(n, seed):
    import torch
    keys = workloads.mix_keys_torch(torch.arange(seed << 40, (seed << 40) + n, device="cuda"))
    return keys, torch.arange(n, dtype=torch.int32, device="cuda") * 3 + 1


def _needles(keys, m, seed, kind):
    """Needles and the position of each in `keys`, -1 for a miss."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n = keys.numel()
    at = torch.randint(0, n, (m,), generator=g, device="cuda")
    if kind == "one":
        at.fill_(n // 3)
    elif kind == "few":
        at = at % 5
    elif kind == "ascending":
        at = torch.sort(keys).indices[torch.sort(at).values]
    elif kind == "misses":
        at.fill_(-1)
    else:
        at[torch.rand(m, generator=g, device="cuda") < 0.4] = -1
    miss = workloads.mix_keys_torch(torch.arange((seed + 77) << 40, ((seed + 77) << 40) + m, device="cuda"))
    return torch.where(at >= 0, keys[at.clamp(min=0)], miss), at


def _check(v, f, vals, at, missing):
    import torch
    hit = at >= 0
    if f is not None:
        assert torch.equal(f, hit.to(torch.uint8))
    if v is not None:
        want = torch.where(hit, vals[at.clamp(min=0)], torch.tensor(missing, dtype=vals.dtype, device="cuda"))
        assert torch.equal(v, want)


def _i32(x):
    return x - (1 << 32) if x >= 1 << 31 else x


SHAPES = [(1 << 22, 1 << 22), ((1 << 22) + 1, 274 * TILE), (1 << 18, 547 * TILE + 1), (3000017, (1 << 23) - 1 + TILE)]


@pytest.mark.parametrize("kind", ["mixed", "one", "few", "ascending", "misses"])
@pytest.mark.parametrize("n,m", SHAPES)
def test_maps_and_comparison_maps(n, m, kind):
    import torch
    announce(f"gpu ordered: n={n} m={m} {kind}")
    keys, vals = _table(n, 1)
    q, at = _needles(keys, m, 2, kind)
    v = torch.empty(m, dtype=torch.int32, device="cuda")
    f = torch.empty(m, dtype=torch.uint8, device="cuda")
    mp = fks.fks_build_u64(keys, vals, 7)
    fks.fks_lookup_u64(mp, q, v, f, missing=MISSING)
    _check(v, f, vals, at, _i32(MISSING))
    f.fill_(9)
    fks.fks_contains_u64(mp, q, f)
    _check(None, f, vals, at, 0)
    for layout in (0, 1):
        s = fks.fks_sorted_build_u64(keys, vals, layout)
        v.fill_(5)
        f.fill_(9)
        fks.fks_sorted_lookup_u64(s, q, v, f, missing=MISSING)
        _check(v, f, vals, at, _i32(MISSING))
        s.destroy()
    mp.destroy()


@pytest.mark.parametrize("n,m", [(1 << 22, 1 << 22), (1 << 18, 547 * TILE - 1)])
def test_64_bit_values(n, m):
    import torch
    announce(f"gpu ordered: 64-bit values n={n} m={m}")
    keys, _ = _table(n, 3)
    vals = workloads.mix_keys_torch(torch.arange(n, device="cuda"))
    q, at = _needles(keys, m, 4, "mixed")
    v = torch.empty(m, dtype=torch.int64, device="cuda")
    f = torch.empty(m, dtype=torch.uint8, device="cuda")
    mp = fks.fks_build_u64_v64(keys, vals, 7)
    fks.fks_lookup_u64_v64(mp, q, v, f, missing=12345678901234)
    _check(v, f, vals, at, 12345678901234)
    v.fill_(0)
    fks.fks_lookup_u64_v64(mp, q, v, missing=12345678901234)
    _check(v, None, vals, at, 12345678901234)
    fks.fks_contains_u64(mp, q, f)
    _check(None, f, vals, at, 0)
    mp.destroy()


@pytest.mark.parametrize("kind", ["mixed", "one map"])
@pytest.mark.parametrize("maps,size,m", [(700, 6007, 1 << 22), (64, 65536, 342 * TILE_IDS + 5), (9000, 450, 700 * TILE_IDS - 1)])
def test_batches(maps, size, m, kind):
    import torch
    announce(f"gpu ordered: batch of {maps} maps of about {size}, m={m} {kind}")
    rng = np.random.default_rng(maps)
    sizes = rng.integers(size // 2, size + 1, size=maps)
    off = np.zeros(maps + 1, np.uint64)
    np.cumsum(sizes, out=off[1:])
    total = int(off[-1])
    keys, vals = _table(total, 5)
    b = fks.fks_build_batch_u64(keys, vals, off, 11)
    q, at = _needles(keys, m, 6, "mixed")
    owner = torch.repeat_interleave(torch.arange(maps, device="cuda"), torch.from_numpy(sizes).cuda())
    ids = torch.where(at >= 0, owner[at.clamp(min=0)], torch.arange(m, device="cuda") % (maps + 3))
    if kind == "one map":
        ids.fill_(maps // 2)
        at = torch.where((at >= 0) & (owner[at.clamp(min=0)] == maps // 2), at, torch.full_like(at, -1))
    ids = ids.to(torch.int32)          # ids from the number of maps on: no such map, every needle absent
    v = torch.empty(m, dtype=torch.int32, device="cuda")
    f = torch.empty(m, dtype=torch.uint8, device="cuda")
    fks.fks_lookup_batch_u64(b, ids, q, v, f, missing=MISSING)
    _check(v, f, vals, at, _i32(MISSING))
    b.destroy()


def test_more_than_one_slice():
    import torch
    n, m = 1 << 20, (1 << 27) + 40 * TILE + 11
    announce(f"gpu ordered: n={n} m={m}")
    keys, vals = _table(n, 1)
    q, at = _needles(keys, m, 2, "mixed")
    v = torch.empty(m, dtype=torch.int32, device="cuda")
    f = torch.empty(m, dtype=torch.uint8, device="cuda")
    mp = fks.fks_build_u64(keys, vals, 7)
    fks.fks_lookup_u64(mp, q, v, f, missing=MISSING)
    _check(v, f, vals, at, _i32(MISSING))
    mp.destroy()


def test_calls_behind_each_other_on_streams():
    """Many calls in flight on three streams: scratch passes from call to call."""
    import torch
    n = m = 1 << 22
    announce("gpu ordered: calls in flight on streams")
    keys, vals = _table(n, 1)
    mp = fks.fks_build_u64(keys, vals, 7)
    qs = [_needles(keys, m, s, "mixed") for s in range(4)]
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    streams = [torch.cuda.Stream() for _ in range(3)]
    outs = []
    for k in range(24):
        st = streams[k % 3]
        with torch.cuda.stream(st):
            v = torch.empty(m, dtype=torch.int32, device="cuda")
            f = torch.empty(m, dtype=torch.uint8, device="cuda")
            fks.fks_lookup_u64(mp, qs[k % 4][0], v, f, missing=MISSING, stream=st)
        outs.append((v, f, k % 4))
    torch.cuda.synchronize()
    for v, f, k in outs:
        _check(v, f, vals, qs[k][1], _i32(MISSING))
    held = free - torch.cuda.mem_get_info()[0] - 24 * 5 * m
    assert held < 8 * 15 * m + (256 << 20)       # a few calls' scratch, not one for each call
    mp.destroy()


def test_capture_and_callers_memory_keep_the_direct_path():
    import torch
    n = m = 1 << 22
    announce("gpu ordered: capture, caller's allocator")
    keys, vals = _table(n, 1)
    q, at = _needles(keys, m, 2, "mixed")
    v = torch.empty(m, dtype=torch.int32, device="cuda")
    f = torch.empty(m, dtype=torch.uint8, device="cuda")
    mp = fks.fks_build_u64(keys, vals, 7, allocator=fks.torch_allocator())
    fks.fks_lookup_u64(mp, q, v, f, missing=MISSING)
    _check(v, f, vals, at, _i32(MISSING))
    mp.destroy()
    mp = fks.fks_build_u64(keys, vals, 7)
    fks.fks_lookup_u64(mp, q, v, f, missing=MISSING)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        fks.fks_lookup_u64(mp, q, v, f, missing=MISSING, stream=torch.cuda.current_stream())
    for k in range(3):
        q2, at2 = _needles(keys, m, 20 + k, "mixed")
        q.copy_(q2)
        v.zero_()
        g.replay()
        torch.cuda.synchronize()
        _check(v, f, vals, at2, _i32(MISSING))
    del g
    mp.destroy()
