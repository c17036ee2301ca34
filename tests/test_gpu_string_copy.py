"""GPU test of the pass that fingerprints strings and copies them into the map: lengths around
its 64-byte words and 16-byte pieces, runs too long to stage, bytes before the first and
after the last string, aligned and unaligned input; the input is overwritten before the
lookups, so that every answer comes from the copy."""
import numpy as np
import pytest

import oracle
from paper_2508_11443_amd import fks
from tests.gpu_util import announce, to_dev

pytestmark = pytest.mark.gpu

LENGTHS = {
    "short": lambda rng, n: rng.integers(0, 18, size=n),
    "around 64": lambda rng, n: rng.integers(60, 69, size=n),
    "mixed": lambda rng, n: np.where(rng.random(n) < 0.03, rng.integers(65, 3000, size=n), rng.integers(0, 65, size=n)),
    "all 64": lambda rng, n: np.full(n, 64),
    "long": lambda rng, n: rng.integers(4000, 9000, size=n),
}


@pytest.mark.parametrize("shift", [0, 1, 4, 15])
@pytest.mark.parametrize("lengths,n,head,tail", [("short", 1000, 0, 0), ("short", 4097, 5, 3), ("around 64", 3001, 0, 100),
                                                 ("mixed", 2000, 16, 0), ("all 64", 640, 33, 0), ("long", 65, 1, 1),
                                                 ("short", 1, 0, 0), ("mixed", 63, 100, 70)])
def test_answers_come_from_the_copy(lengths, n, head, tail, shift):
    import torch
    announce(f"gpu string copy: {lengths} n={n} head={head} tail={tail} shift={shift}")
    rng = np.random.default_rng(n + head)
    lens = LENGTHS[lengths](rng, n)
    if lengths in ("short", "mixed"):
        lens = np.maximum(lens, 5)      # room for a number that makes the strings distinct
        lens[0] = 0
    off = np.zeros(n + 1, np.int64)
    off[0] = head
    np.cumsum(lens, out=off[1:])
    off[1:] += head
    data = rng.integers(0, 256, size=int(off[-1]) + tail, dtype=np.uint8)
    for i in range(n):
        k = min(4, int(lens[i]))
        data[off[i]: off[i] + k] = np.frombuffer(int(i * 2654435761 % (1 << 32)).to_bytes(4, "little"), np.uint8)[:k]
    vals = np.arange(n, dtype=np.uint32) * 7 + 1
    room = torch.zeros(data.size + 64, dtype=torch.uint8, device="cuda")
    base = (16 - room.data_ptr() % 16) % 16 + shift
    d_data = room[base: base + data.size]
    d_data.copy_(to_dev(data))
    d_off = to_dev(off)
    m = fks.fks_build_bytes(d_off, d_data, to_dev(vals), 99 + shift)
    ref = oracle.build_bytes(off, data, vals, 99 + shift)
    h, s, _ = fks.fks_export(m)
    rh, rs = ref.export()
    assert (h == rh).all() and (s == rs).all()
    q_off, q_data = to_dev(off), to_dev(data)
    room.fill_(0)
    d_off.fill_(0)
    v = torch.empty(n, dtype=torch.int32, device="cuda")
    f = torch.empty(n, dtype=torch.uint8, device="cuda")
    fks.fks_lookup_bytes(m, q_off, q_data, v, f, missing=0)
    assert bool(f.all()) and (v.cpu().numpy().view(np.uint32) == vals).all()
    # the last byte of every string changed: only the empty string is still there
    other = data.copy()
    has = lens > 0
    other[(off[1:] - 1)[has]] ^= 0x5A
    fks.fks_lookup_bytes(m, q_off, to_dev(other), v, f, missing=0)
    assert (f.cpu().numpy() == (~has).astype(np.uint8)).all()
    m.destroy()
