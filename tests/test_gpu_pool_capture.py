"""GPU test of the library's own memory beside a graph capture: while one thread captures a stream in
the default mode, which refuses what could disturb the capture, another asks lookups that take and
return scratch on its own stream; the capture ends well and its graph replays right."""
import threading

import pytest

from paper_2508_11443_amd import fks, workloads
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


def test_other_threads_lookups_during_a_capture():
    import torch
    n = m = 1 << 22
    announce("gpu pool capture: lookups in another thread")
    keys = workloads.mix_keys_torch(torch.arange(n, device="cuda"))
    vals = torch.arange(n, dtype=torch.int32, device="cuda")
    mp = fks.fks_build_u64(keys, vals, 7)
    side = torch.cuda.Stream()
    outs = [(torch.empty(m, dtype=torch.int32, device="cuda"), torch.empty(m, dtype=torch.uint8, device="cuda"))
            for _ in range(3)]
    qs = [keys[torch.randperm(n, device="cuda")].contiguous() for _ in range(3)]
    x = torch.arange(1000, dtype=torch.int64, device="cuda")
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    go, done, errors = threading.Event(), threading.Event(), []

    def work():
        try:
            go.wait(30)
            for _ in range(3):         # the first takes memory, the others take what is on its way back
                for q, (v, f) in zip(qs, outs):
                    fks.fks_lookup_u64(mp, q, v, f, stream=side)
        except BaseException as e:   # reported by the main thread
            errors.append(e)
        finally:
            done.set()

    t = threading.Thread(target=work)
    t.start()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y.add_(x)
        go.set()
        assert done.wait(60)
        y.add_(x)
    t.join()
    if errors:
        raise errors[0]
    for k in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, 2 * x)
    for q, (v, f) in zip(qs, outs):
        assert bool(f.all()) and torch.equal(keys[v.long()], q)
    del g
    mp.destroy()
