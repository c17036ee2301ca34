"""GPU test of the library's own device memory: maps of mixed sizes are built, asked and released
in loops, on the null stream, on side streams and from several threads at once, so that blocks
are split, merged and handed from stream to stream; every answer is checked, and the memory held
for reuse stays within its bound."""
import threading

import numpy as np
import pytest

from paper_2508_11443_amd import fks, workloads
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


def _loop(torch, stream, rounds, seed, sizes, errors):
    """Builds and releases maps over `sizes` in turn, three alive at a time; the answers of a
    map are compared after its memory may have been handed on."""
    try:
        rng = np.random.default_rng(seed)
        alive, checks = [], []
        with torch.cuda.stream(stream):
            for k in range(rounds):
                n = int(rng.choice(sizes))
                idx = torch.arange(seed << 40, (seed << 40) + n, device="cuda")
                keys = workloads.mix_keys_torch(idx + (k << 30))
                vals = torch.arange(n, dtype=torch.int32, device="cuda")
                m = fks.fks_build_u64(keys, vals, seed + k, stream=stream)
                q = torch.cat([keys, keys ^ 1])
                v = torch.empty(2 * n, dtype=torch.int32, device="cuda")
                f = torch.empty(2 * n, dtype=torch.uint8, device="cuda")
                fks.fks_lookup_u64(m, q, v, f, stream=stream)
                alive.append(m)
                checks.append((keys, vals, v, f))
                if len(alive) == 3:
                    stream.synchronize()   # a map is released after its last lookup
                    alive.pop(int(rng.integers(3))).destroy()
            stream.synchronize()
            for keys, vals, v, f in checks:
                n = vals.numel()
                assert bool((f[:n] == 1).all()) and bool((v[:n] == vals).all())
                assert not bool(f[n:].any())
        for m in alive:
            m.destroy()
    except BaseException as e:   # reported by the main thread
        errors.append(e)


@pytest.mark.parametrize("threads", [1, 4])
def test_blocks_pass_between_maps_and_streams(threads):
    import torch
    announce(f"gpu pool: {threads} thread(s)")
    errors = []
    sizes = [1, 1000, 5000, 70000, 300007, 1 << 20]
    _loop(torch, torch.cuda.current_stream(), 12, 1, sizes, errors)
    runs = [threading.Thread(target=_loop, args=(torch, torch.cuda.Stream(), 12, 2 + t, sizes, errors))
            for t in range(threads)]
    for r in runs:
        r.start()
    for r in runs:
        r.join()
    if errors:
        raise errors[0]


def test_memory_kept_for_reuse_is_bounded():
    """Maps of ever larger sizes: what stays reserved once they are gone is at most an eighth of
    the device, give or take the largest segment."""
    import torch
    announce("gpu pool: bound on the memory kept")
    torch.cuda.synchronize()
    total = torch.cuda.mem_get_info()[1]
    before = torch.cuda.mem_get_info()[0]
    for lg in range(20, 26):
        n = 1 << lg
        keys = workloads.mix_keys_torch(torch.arange(n, device="cuda"))
        m = fks.fks_build_u64(keys, torch.arange(n, dtype=torch.int32, device="cuda"), lg)
        m.destroy()
        del keys
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    assert before - torch.cuda.mem_get_info()[0] <= total // 8 + (4 << 30)
