"""GPU test of the fused final pass's look-back where a predecessor's sum is late: a build that
polls for no sum at all, or once, takes it from that partition's records instead, and writes the
oracle's bytes, also where the pass runs a second time into a larger table or rejects the
attempt; builds on streams side by side, each too large for the chip alone, find all their keys."""
import contextlib
import ctypes
import threading

import numpy as np
import pytest

import oracle
from paper_2508_11443_amd import fks, workloads
from tests.gpu_util import announce, to_dev
from tests.test_gpu_single import assert_same_table, skewed_keys

pytestmark = pytest.mark.gpu

DEFAULT = 128


@contextlib.contextmanager
def patience(polls):
    """Polls of a predecessor's word in this thread's builds (the library's internal setting)."""
    import torch  # noqa: F401  (its HIP runtime first: the library shares it)
    f = getattr(fks.library(), "_ZN3fks13part_patienceEj")
    f.argtypes, f.restype = [ctypes.c_uint32], None
    f(polls)
    try:
        yield
    finally:
        f(DEFAULT)


@pytest.mark.parametrize("polls", [0, 1])
@pytest.mark.parametrize("n", [1024, 1025, 70007, 131073, 600011])
def test_integer_maps(n, polls):
    announce(f"gpu look-back: n={n} polls={polls}")
    keys = workloads.unique_u64(n, n, dense_fraction=0.5)
    vals = np.arange(n, dtype=np.uint32)
    with patience(polls):
        m = fks.fks_build_u64(to_dev(keys), to_dev(vals), n)
        w = fks.fks_build_u64_v64(to_dev(keys), to_dev(vals.astype(np.uint64) << np.uint64(31)), n)
    assert_same_table(m, oracle.build_u64(keys, vals, n))
    assert (fks.fks_export(w)[0] == fks.fks_export(m)[0]).all()
    f = to_dev(np.zeros(n, np.uint8))
    fks.fks_contains_u64(w, to_dev(keys), f)
    assert bool(f.all())


@pytest.mark.parametrize("polls", [0, 1, DEFAULT])
@pytest.mark.parametrize("n,per_bucket,c", [(6000, 5, 8), (100003, 5, 8), (600011, 5, 8)])
def test_second_pass_into_a_larger_table(n, per_bucket, c, polls):
    """S near 5n: above the 4n cells taken at first."""
    announce(f"gpu look-back: S near {per_bucket}n, n={n} polls={polls}")
    keys = skewed_keys(n, 0x2B + n, per_bucket, n)
    vals = np.arange(n, dtype=np.uint32)
    ref = oracle.build_u64(keys, vals, 0x2B + n, c=c)
    assert ref.r == 0 and ref.S > 4 * n
    with patience(polls):
        m = fks.fks_build_u64(to_dev(keys), to_dev(vals), 0x2B + n, c=c)
    assert_same_table(m, ref)


@pytest.mark.parametrize("case", ["oversize", "space"])
def test_rejected_attempt(case):
    n, seed = 50000, 0x1DD + len(case)
    announce(f"gpu look-back: first attempt rejected ({case})")
    if case == "oversize":
        keys, kw = skewed_keys(n, seed, 1, 77, big=16), {}
    else:
        keys, kw = skewed_keys(n, seed, 3, 78), {"c": 2}
    vals = np.arange(n, dtype=np.uint32)
    ref = oracle.build_u64(keys, vals, seed, **kw)
    assert ref.r >= 1
    with patience(0):
        m = fks.fks_build_u64(to_dev(keys), to_dev(vals), seed, **kw)
    assert_same_table(m, ref)


def test_strings():
    n = 70007
    announce("gpu look-back: strings")
    off, data = workloads.random_strings(n, 5, 4, 64)
    vals = np.arange(n, dtype=np.uint32)
    with patience(0):
        m = fks.fks_build_bytes(to_dev(off), to_dev(data), to_dev(vals), 9)
    assert_same_table(m, oracle.build_bytes(off, data, vals, 9))


def test_batch():
    announce("gpu look-back: batch of wide maps")
    sizes = [4096, 65536, 5121, 300, 12289, 65535]
    off = np.zeros(len(sizes) + 1, np.uint64)
    np.cumsum(np.array(sizes, np.uint64), out=off[1:])
    keys = workloads.unique_u64(int(off[-1]), 78, dense_fraction=0.4)
    vals = np.arange(keys.size, dtype=np.uint32)
    with patience(0):
        b = fks.fks_build_batch_u64(to_dev(keys), to_dev(vals), off, 4243)
    for m in range(len(sizes)):
        lo, hi = int(off[m]), int(off[m + 1])
        h, s = fks.fks_batch_export(b, m)[:2]
        rh, rs = oracle.build_u64(keys[lo:hi], vals[lo:hi], oracle.batch_seed(4243, m)).export()
        assert (h == rh).all() and (s == rs).all(), m
    b.destroy()


def test_large_builds_side_by_side():
    import torch
    n = 6_000_003
    announce("gpu look-back: two large builds at a time")
    errors = []

    def work(t, stream):
        try:
            with torch.cuda.stream(stream):
                keys = workloads.mix_keys_torch(torch.arange(t << 40, (t << 40) + n, device="cuda"))
                vals = torch.arange(n, dtype=torch.int32, device="cuda")
                v = torch.empty_like(vals)
                f = torch.empty(n, dtype=torch.uint8, device="cuda")
                for k in range(6):
                    m = fks.fks_build_u64(keys, vals, 100 * t + k, stream=stream)
                    fks.fks_lookup_u64(m, keys, v, f, stream=stream)
                    stream.synchronize()
                    assert bool(f.all()) and torch.equal(v, vals)
                    m.destroy()
        except BaseException as e:   # reported by the main thread
            errors.append(e)

    runs = [threading.Thread(target=work, args=(t, torch.cuda.Stream())) for t in range(2)]
    for r in runs:
        r.start()
    for r in runs:
        r.join()
    if errors:
        raise errors[0]
