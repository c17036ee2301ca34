"""Measured cases: what programs have this library do, through its public entry points.

A case is a plain dict.  ``listed()`` gives the cases that are always timed, ``draw(rng)`` one
more of the same ranges, ``prepare(case, seed)`` the inputs and long-lived objects a program
has in hand before the call (on the GPU), ``run(state)`` one pass, ``work(case)`` the bytes a
pass cannot do without, ``exact(case, seed)`` the answers of dictionary semantics, computed
with plain torch from the way the inputs were made.

Keys are distinct by construction (a seeded bijection of a counter), as the sizes call for
inputs made on the device; lookups are answered into buffers that the program keeps.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2508_11443_amd import fks

MISSING = 0xFFFFFFFF
STRING_RANGES = {"4-64": (4, 64), "5-25": (5, 25)}


# ---- the cases ------------------------------------------------------------------------

def listed():
    return [
        # a request against a resident dictionary, too small to fill the chip: launch and latency
        {"name": "lookup_small", "kind": "lookup", "n": 1 << 16, "m": 1000, "dense": 0.0, "hits": 0.5, "op": "lookup"},
        # the small map: built, asked once for as many needles, released (launches, one host wait)
        {"name": "step_small", "kind": "step", "n": 1 << 16, "m": 1 << 16, "dense": 0.0, "hits": 0.5, "op": "lookup"},
        # the paper's own benchmark shape: 10^7 uniform keys, every key looked up once
        {"name": "step_paper", "kind": "step", "n": 10_000_000, "m": 10_000_000, "dense": 0.0, "hits": 1.0,
         "op": "lookup"},
        # the benchmark's step: 2^26 keys, half of them one dense run, 2^26 needles at 50 % hits
        {"name": "step_large", "kind": "step", "n": 1 << 26, "m": 1 << 26, "dense": 0.5, "hits": 0.5, "op": "lookup"},
        # 64-bit values (pointers, offsets) at an odd size
        {"name": "v64_mid", "kind": "v64", "n": 3_000_017, "m": 1_500_001, "dense": 0.0, "hits": 0.75},
        # string keys of 4-64 bytes, the benchmark's size
        {"name": "strings", "kind": "strings", "n": 1 << 22, "m": 1 << 22, "lengths": "4-64", "hits": 0.5,
         "op": "lookup"},
        # the constructor that takes repeated keys: every key about twice
        {"name": "from_array", "kind": "from_array", "n": 1 << 23, "m": 1 << 20, "distinct": 0.5, "hits": 0.5},
        # thousands of small dictionaries built at once, needles spread over them
        {"name": "batch", "kind": "batch", "maps": 4096, "hi": 1 << 16, "m": 1 << 24, "hits": 0.75},
        # the values of a resident map changed and folded, some of them looked up
        {"name": "values", "kind": "values", "n": 1 << 24, "m": 2_200_003},
        # the comparison maps of the paper: sorted array with binary search, Eytzinger order
        {"name": "sorted", "kind": "sorted", "n": 1 << 24, "m": 1 << 24, "dense": 0.5, "hits": 0.5, "layout": 0},
        {"name": "eytzinger", "kind": "sorted", "n": 10_000_000, "m": 10_000_000, "dense": 0.0, "hits": 1.0,
         "layout": 1},
        # a burst of requests to the serving loop: lookups against resident maps while two maps are built
        {"name": "serve_burst", "kind": "serve", "resident": 1 << 20, "lookups": 24, "m": 1 << 16, "build": 1 << 18},
    ]


def _size(rng, lo, hi):
    """A size in [lo, hi], its logarithm uniform; odd sizes are as likely as even ones."""
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _asked(rng):
    """The question and its share of hits (membership is asked where some keys are absent)."""
    op = rng.choice(["lookup", "contains"])
    return {"op": op, "hits": rng.choice([0.25, 0.5, 1.0] if op == "lookup" else [0.25, 0.5, 0.75])}


def draw(rng):
    kind = rng.choice(["lookup", "step", "step", "v64", "strings", "from_array", "batch", "values", "sorted",
                       "sorted", "serve"])
    if kind == "lookup":
        return {"kind": kind, "n": _size(rng, 1 << 10, 1 << 24), "m": _size(rng, 1 << 8, 1 << 20),
                "dense": rng.choice([0.0, 0.5]), **_asked(rng)}
    if kind == "step":
        return {"kind": kind, "n": _size(rng, 1 << 8, 1 << 26), "m": _size(rng, 1 << 8, 1 << 26),
                "dense": rng.choice([0.0, 0.5]), **_asked(rng)}
    if kind == "v64":
        return {"kind": kind, "n": _size(rng, 1 << 10, 1 << 24), "m": _size(rng, 1 << 8, 1 << 24),
                "dense": rng.choice([0.0, 0.5]), "hits": rng.choice([0.5, 0.75, 1.0])}
    if kind == "strings":
        return {"kind": kind, "n": _size(rng, 1 << 10, 1 << 22), "m": _size(rng, 1 << 8, 1 << 22),
                "lengths": rng.choice(sorted(STRING_RANGES)), **_asked(rng)}
    if kind == "from_array":
        return {"kind": kind, "n": _size(rng, 1 << 10, 1 << 23), "m": _size(rng, 1 << 8, 1 << 22),
                "distinct": rng.choice([0.01, 0.5, 0.9]), "hits": 0.5}
    if kind == "batch":
        return {"kind": kind, "maps": _size(rng, 16, 1 << 12), "hi": _size(rng, 1 << 8, 1 << 16),
                "m": _size(rng, 1 << 12, 1 << 24), "hits": rng.choice([0.5, 0.75])}
    if kind == "values":
        return {"kind": kind, "n": _size(rng, 1 << 10, 1 << 25), "m": _size(rng, 1 << 10, 1 << 22)}
    if kind == "sorted":
        return {"kind": kind, "n": _size(rng, 1 << 10, 1 << 24), "m": _size(rng, 1 << 8, 1 << 23),
                "dense": rng.choice([0.0, 0.5]), "hits": rng.choice([0.5, 1.0]), "layout": rng.choice([0, 1])}
    return {"kind": "serve", "resident": _size(rng, 1 << 12, 1 << 22), "lookups": rng.randint(4, 32),
            "m": _size(rng, 1 << 8, 1 << 18), "build": _size(rng, 1 << 10, 1 << 20)}


# ---- inputs -----------------------------------------------------------------------------

def _device():
    return torch.device("cuda", torch.cuda.current_device())


class _Maker:
    """Seeded inputs on the device: a bijection of 64-bit counters, and a generator."""

    def __init__(self, seed):
        self.dev = _device()
        rng = random.Random(0x5EED ^ (seed * 0x9E3779B97F4A7C15))
        self.rng = rng
        self.mul = [(rng.getrandbits(64) | 1) - (1 << 63) for _ in range(2)]
        self.mul = [a | 1 for a in self.mul]
        self.add = rng.getrandbits(63)
        self.gen = torch.Generator(device=self.dev)
        self.gen.manual_seed(rng.getrandbits(62))
        self.map_seed = rng.getrandbits(63)

    def spread(self, idx):
        """Distinct 64-bit words for distinct counters."""
        x = idx + self.add
        for a, s in zip(self.mul, (32, 29)):
            x = x * a
            x = x ^ ((x >> s) & ((1 << (64 - s)) - 1))
        return x

    def arange(self, lo, hi):
        return torch.arange(lo, hi, dtype=torch.int64, device=self.dev)

    def perm(self, n):
        return torch.randperm(n, generator=self.gen, device=self.dev)

    def below(self, hi, count):
        return torch.randint(0, hi, (count,), generator=self.gen, device=self.dev)

    def pick(self, n, count):
        """Positions in [0, n): without repeats where that is possible."""
        return self.perm(n)[:count] if count <= n else self.below(n, count)

    def keys_and_misses(self, n, dense, misses):
        """n distinct keys in random order (a share of them one run of consecutive integers)
        and `misses` words that are not keys."""
        nd = int(n * dense)
        u = self.spread(self.arange(0, n - nd + misses))
        while nd:
            base = self.rng.getrandbits(62)
            if not bool(((u >= base) & (u < base + nd)).any()):
                break
        keys = u[: n - nd]
        if nd:
            keys = torch.cat([keys, self.arange(base, base + nd)])
        return keys[self.perm(n)], u[n - nd:]

    def needles(self, keys, misses, hits_at):
        """Needles in random order: keys[hits_at] and the misses; the position in `keys` of
        each needle, -1 for a miss."""
        q = torch.cat([keys[hits_at], misses])
        at = torch.cat([hits_at, torch.full((misses.numel(),), -1, dtype=torch.int64, device=self.dev)])
        p = self.perm(q.numel())
        return q[p].contiguous(), at[p]


def _u32(x):
    return x.to(torch.int32)


def _outputs(m, dev, wide=False):
    return (torch.empty(m, dtype=torch.int64 if wide else torch.int32, device=dev),
            torch.empty(m, dtype=torch.uint8, device=dev))


def _answers(vals, at, missing):
    """What lookups answer: the value of the key at each position, `missing` for -1."""
    found = at >= 0
    none = torch.tensor(missing, dtype=vals.dtype, device=vals.device)
    return torch.where(found, vals[at.clamp(min=0)], none), found.to(torch.uint8)


def _integer_inputs(case, seed):
    mk = _Maker(seed)
    n, m = case["n"], case["m"]
    nh = int(round(m * case["hits"]))
    keys, misses = mk.keys_and_misses(n, case["dense"], m - nh)
    vals = mk.spread(mk.arange(0, n)) if case["kind"] == "v64" else _u32(mk.arange(0, n))
    q, at = mk.needles(keys, misses, mk.pick(n, nh))
    return mk, keys, vals, q, at


def _strings(mk, count, lo, hi):
    """`count` distinct lowercase strings with lengths uniform in [lo, hi], as (offsets, bytes)."""
    dev = mk.dev
    lens = torch.randint(lo, hi + 1, (count,), generator=mk.gen, device=dev)
    order = torch.argsort(lens, stable=True)
    per = torch.bincount(lens, minlength=hi + 1)
    starts = torch.cumsum(per, 0) - per
    rank = torch.empty(count, dtype=torch.int64, device=dev)
    rank[order] = mk.arange(0, count) - starts[lens[order]]     # place among the strings of its length
    # the first min(length, 12) letters spell a permutation of the rank, the rest are random
    digits = lens.clamp(max=12)
    space = torch.tensor([26 ** k for k in range(13)], dtype=torch.int64, device=dev)[digits]
    mult = 26 * mk.rng.getrandbits(33) + 17                     # prime to 26
    code = (rank * mult + lens * mk.rng.getrandbits(48) + mk.rng.getrandbits(56)) % space
    off = torch.zeros(count + 1, dtype=torch.int64, device=dev)
    torch.cumsum(lens, 0, out=off[1:])
    total = int(off[-1])
    data = torch.randint(ord("a"), ord("z") + 1, (total,), generator=mk.gen, device=dev, dtype=torch.uint8)
    for p in range(min(12, hi)):
        has = torch.nonzero(lens > p).squeeze(1)
        data[off[has] + p] = (code[has] // 26 ** p % 26 + ord("a")).to(torch.uint8)
    return off, data


def _take_strings(off, data, idx):
    lens = off[idx + 1] - off[idx]
    out = torch.zeros(idx.numel() + 1, dtype=torch.int64, device=off.device)
    torch.cumsum(lens, 0, out=out[1:])
    src = torch.repeat_interleave(off[idx] - out[:-1], lens)
    return out, data[src + torch.arange(int(out[-1]), device=off.device)]


def _string_inputs(case, seed):
    mk = _Maker(seed)
    n, m = case["n"], case["m"]
    lo, hi = STRING_RANGES[case["lengths"]]
    nh = int(round(m * case["hits"]))
    off, data = _strings(mk, n + m - nh, lo, hi)
    idx = torch.cat([mk.pick(n, nh), mk.arange(n, n + m - nh)])[mk.perm(m)]
    at = torch.where(idx < n, idx, torch.full_like(idx, -1))
    end = int(off[n])
    return mk, (off[: n + 1].clone(), data[:end].clone()), _u32(mk.arange(0, n)), _take_strings(off, data, idx), at


def _repeated_inputs(case, seed):
    mk = _Maker(seed)
    u, m = case["n"], case["m"]
    distinct = max(1, int(u * case["distinct"]))
    which = mk.below(distinct, u)
    vals = _u32(mk.arange(0, u))
    nh = int(round(m * case["hits"]))
    at = torch.cat([mk.below(u, nh), torch.full((m - nh,), -1, dtype=torch.int64, device=mk.dev)])
    miss = mk.spread(mk.arange(distinct, distinct + m - nh))
    keys = mk.spread(which)
    q = torch.cat([keys[at[:nh]], miss])
    p = mk.perm(m)
    return mk, keys, which, vals, q[p].contiguous(), at[p]


def _batch_inputs(case, seed):
    mk = _Maker(seed)
    rng = np.random.Generator(np.random.PCG64(seed))
    M, m = case["maps"], case["m"]
    lo, hi = 16, case["hi"]
    sizes = np.clip(np.exp(rng.uniform(np.log(lo), np.log(hi), size=M)).astype(np.int64), lo, hi)
    offsets = np.zeros(M + 1, np.int64)
    np.cumsum(sizes, out=offsets[1:])
    total = int(offsets[-1])
    d_off, d_size = torch.from_numpy(offsets).to(mk.dev), torch.from_numpy(sizes).to(mk.dev)
    keys = mk.spread(mk.arange(0, total))
    vals = _u32(mk.arange(0, total) - torch.repeat_interleave(d_off[:-1], d_size))
    ids = mk.below(M, m)
    hit = torch.rand(m, generator=mk.gen, device=mk.dev) < case["hits"]
    pick = (torch.rand(m, generator=mk.gen, device=mk.dev, dtype=torch.float64) * d_size[ids]).to(torch.int64)
    at = torch.where(hit, d_off[ids] + pick, torch.full_like(ids, -1))
    q = torch.where(hit, keys[at.clamp(min=0)], mk.spread(mk.arange(total, total + m)))
    return mk, keys, vals, offsets.astype(np.uint64), _u32(ids), q, at


def _value_inputs(case, seed):
    mk = _Maker(seed)
    n, m = case["n"], case["m"]
    keys, _ = mk.keys_and_misses(n, 0.0, 0)
    vals = _u32(mk.spread(mk.arange(0, n)) & 0xFFFFFFFF)
    at = mk.pick(n, m)
    a, b = mk.rng.getrandbits(32) | 1, mk.rng.getrandbits(32)
    return mk, keys, vals, keys[at].contiguous(), at, a, b


def _serve_inputs(case, seed):
    """Keys of two resident maps and two that are built, and a burst of lookup batches whose
    sizes spread over a factor of 64 below the largest."""
    mk = _Maker(seed)
    keys, vals = [], []
    for k, n in enumerate((case["resident"], max(256, case["resident"] // 4), case["build"],
                           max(256, case["build"] // 4))):
        keys.append(mk.spread(mk.arange(k << 40, (k << 40) + n)))
        vals.append(_u32(mk.arange(0, n)))
    asks = []
    for k in range(case["lookups"]):
        m = max(16, int(case["m"] * 64.0 ** -(k * 0.618 % 1.0)))
        of = k % 2
        nh = m // 2
        misses = mk.spread(mk.arange((8 + k) << 40, ((8 + k) << 40) + m - nh))
        q, at = mk.needles(keys[of], misses, mk.pick(keys[of].numel(), min(nh, m)))
        asks.append((of, q, at))
    return mk, keys, vals, asks


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("lookup", "step", "v64", "sorted"):
        mk, keys, vals, q, _ = _integer_inputs(case, seed)
        v, f = _outputs(q.numel(), mk.dev, wide=kind == "v64")
        state = dict(case=case, keys=keys, vals=vals, q=q, v=v, f=f, seed=mk.map_seed)
        if kind == "lookup":
            state["map"] = fks.fks_build_u64(keys, vals, mk.map_seed)
        return state
    if kind == "strings":
        mk, (off, data), vals, (qoff, qdata), _ = _string_inputs(case, seed)
        v, f = _outputs(qoff.numel() - 1, mk.dev)
        return dict(case=case, off=off, data=data, vals=vals, qoff=qoff, qdata=qdata, v=v, f=f, seed=mk.map_seed)
    if kind == "from_array":
        mk, keys, _, vals, q, _ = _repeated_inputs(case, seed)
        v, f = _outputs(q.numel(), mk.dev)
        return dict(case=case, keys=keys, vals=vals, q=q, v=v, f=f, seed=mk.map_seed)
    if kind == "batch":
        mk, keys, vals, offsets, ids, q, _ = _batch_inputs(case, seed)
        v, f = _outputs(q.numel(), mk.dev)
        return dict(case=case, keys=keys, vals=vals, offsets=offsets, ids=ids, q=q, v=v, f=f, seed=mk.map_seed)
    if kind == "values":
        mk, keys, vals, q, _, a, b = _value_inputs(case, seed)
        v, f = _outputs(q.numel(), mk.dev)
        return dict(case=case, map=fks.fks_build_u64(keys, vals, mk.map_seed), q=q, v=v, f=f, a=a, b=b,
                    total=torch.zeros(1, dtype=torch.int64, device=mk.dev))
    mk, keys, vals, asks = _serve_inputs(case, seed)
    server = fks.FksServer(1 << 30)
    ids = [server.submit_build(keys[k], vals[k], mk.map_seed + k)[1] for k in range(2)]
    server.wait_all()
    asks = [(ids[of], q) + _outputs(q.numel(), mk.dev) for of, q, _ in asks]
    return dict(case=case, server=server, asks=asks, seed=mk.map_seed,
                builds=[(keys[k], vals[k]) for k in (2, 3)])


# ---- one pass -----------------------------------------------------------------------------

def _ask(s, m):
    if s["case"]["op"] == "contains":
        fks.fks_contains_u64(m, s["q"], s["f"])
        return [s["f"]]
    fks.fks_lookup_u64(m, s["q"], s["v"], s["f"], missing=MISSING)
    return [s["v"], s["f"]]


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "lookup":
        return _ask(s, s["map"])
    if kind == "step":
        m = fks.fks_build_u64(s["keys"], s["vals"], s["seed"])
        out = _ask(s, m)
        m.destroy()
        return out
    if kind == "v64":
        m = fks.fks_build_u64_v64(s["keys"], s["vals"], s["seed"])
        fks.fks_lookup_u64_v64(m, s["q"], s["v"], s["f"])
        m.destroy()
        return [s["v"], s["f"]]
    if kind == "strings":
        m = fks.fks_build_bytes(s["off"], s["data"], s["vals"], s["seed"])
        if case["op"] == "contains":
            fks.fks_contains_bytes(m, s["qoff"], s["qdata"], s["f"])
        else:
            fks.fks_lookup_bytes(m, s["qoff"], s["qdata"], s["v"], s["f"], missing=MISSING)
        m.destroy()
        return [s["f"]] if case["op"] == "contains" else [s["v"], s["f"]]
    if kind == "from_array":
        m = fks.fks_build_u64_from_array(s["keys"], s["vals"], s["seed"])
        fks.fks_lookup_u64(m, s["q"], s["v"], s["f"], missing=MISSING)
        m.destroy()
        return [s["v"], s["f"]]
    if kind == "batch":
        b = fks.fks_build_batch_u64(s["keys"], s["vals"], s["offsets"], s["seed"])
        fks.fks_lookup_batch_u64(b, s["ids"], s["q"], s["v"], s["f"], missing=MISSING)
        b.destroy()
        return [s["v"], s["f"]]
    if kind == "values":
        m = fks.fks_map_values(s["map"], fks.FKS_VOP_AFFINE, s["a"], s["b"])
        fks.fks_reduce_values(m, fks.FKS_VRED_SUM, out=s["total"])
        fks.fks_lookup_u64(m, s["q"], s["v"], s["f"], missing=MISSING)
        m.destroy()
        return [s["v"], s["f"], s["total"]]
    if kind == "sorted":
        m = fks.fks_sorted_build_u64(s["keys"], s["vals"], case["layout"])
        fks.fks_sorted_lookup_u64(m, s["q"], s["v"], s["f"], missing=MISSING)
        m.destroy()
        return [s["v"], s["f"]]
    server = s["server"]
    for k, (keys, vals) in enumerate(s["builds"]):
        server.submit_build(keys, vals, s["seed"] + 2 + k)
    for map_id, q, v, f in s["asks"]:
        server.submit_lookup(map_id, q, v, f, missing=MISSING)
    server.wait_all()
    return [x for _, _, v, f in s["asks"] for x in (v, f)]


# ---- the least bytes of a pass ---------------------------------------------------------------

# per key of a table: two bytes of bucket header, and about two 16-byte cells
TABLE = 2 + 2 * 16


def _lookups(m, hits, value=4, out_value=4, found=1):
    """Needle in, header record, the cell of a hit, the answer out."""
    return m * (8 + 16 + 16 * hits + out_value * (value > 0) + found)


def work(case):
    kind, n, m = case["kind"], case.get("n", 0), case.get("m", 0)
    b = 0.0
    if kind in ("lookup", "step"):
        b = _lookups(m, case["hits"], 4 if case["op"] == "lookup" else 0)
        if kind == "step":
            b += n * (12 + TABLE)
    elif kind == "v64":
        b = n * (16 + TABLE) + _lookups(m, case["hits"], 8, 8)
    elif kind == "strings":
        lo, hi = STRING_RANGES[case["lengths"]]
        mean = (lo + hi) / 2
        # the map keeps a copy of its keys' bytes and offsets; a hit reads the stored key again
        b = n * (2 * (8 + mean) + 4 + TABLE) + _lookups(m, case["hits"]) + m * mean + m * case["hits"] * (16 + mean)
    elif kind == "from_array":
        b = n * 12 + n * min(1.0, case["distinct"]) * TABLE + _lookups(m, case["hits"])
    elif kind == "batch":
        total = case["maps"] * (case["hi"] - 16) / math.log(case["hi"] / 16) if case["hi"] > 16 else case["maps"] * 16
        b = total * (12 + TABLE) + _lookups(m, case["hits"]) + 4 * m
    elif kind == "values":
        b = n * (2 * TABLE) + n * TABLE + _lookups(m, 1.0)
    elif kind == "sorted":
        b = n * 24 + m * (8 + 8 + 5) + m * case["hits"] * 4
    else:
        each = case["m"] * (63 / 64) / math.log(64)
        b = case["build"] * 1.25 * (12 + TABLE) + case["lookups"] * _lookups(each, 0.5)
    return {"bytes": float(b), "flops": 0.0}


# ---- the answers of dictionary semantics -------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind in ("lookup", "step", "v64", "sorted"):
        _, _, vals, _, at = _integer_inputs(case, seed)
        v, f = _answers(vals, at, -1)
        return [f] if case.get("op") == "contains" else [v, f]
    if kind == "strings":
        _, _, vals, _, at = _string_inputs(case, seed)
        v, f = _answers(vals, at, -1)
        return [f] if case["op"] == "contains" else [v, f]
    if kind == "from_array":
        mk, _, which, vals, _, at = _repeated_inputs(case, seed)
        u = which.numel()
        first = torch.full((int(which.max()) + 1,), u, dtype=torch.int64, device=mk.dev)
        first.scatter_reduce_(0, which, mk.arange(0, u), "amin")
        kept = first[which[at.clamp(min=0)]]       # a repeated key keeps its first occurrence's value
        return list(_answers(vals, torch.where(at >= 0, kept, at), -1))
    if kind == "batch":
        _, _, vals, _, _, _, at = _batch_inputs(case, seed)
        return list(_answers(vals, at, -1))
    if kind == "values":
        _, _, vals, _, at, a, b = _value_inputs(case, seed)
        x = vals.to(torch.int64) & 0xFFFFFFFF
        x = ((x & 0xFFFF) * a + (((x >> 16) * a & 0xFFFF) << 16) + b) & 0xFFFFFFFF
        v, f = _answers(_u32(x), at, -1)
        return [v, f, x.sum().reshape(1)]
    _, _, vals, asks = _serve_inputs(case, seed)
    return [x for of, _, at in asks for x in _answers(vals[of], at, -1)]
