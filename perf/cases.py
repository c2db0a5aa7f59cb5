"""The work a program hands to the library, as measurable cases.

A case is a dict of plain values.  `prepare` makes what a program holds
before the call (device tensors, offsets, a server handle), `run` is one pass
through the public entry points, `work` the bytes a pass cannot do without,
`exact` the same outputs from a plain torch sort.

The sorts work in place, so a pass copies the caller's unsorted arrays into
its working arrays first, as a program does that keeps its input; every pass
then sorts unsorted data.  Keys are 32- or 64-bit patterns held in int32 or
int64 tensors (the order is unsigned); values are 4-byte indexes, as for an
argsort.  The distributions are those of the library's generators: uniform,
the AND of k uniform words, a constant top byte, a 16-key Zipf dictionary
and, for 64-bit keys, keys that vary in some of their bytes only.
"""
import math

import numpy as np
import torch

import paper_1008_2849_amd as rts

DEV = "cuda"
SIGN64 = -(1 << 63)


def listed():
    return [
        # a small lookup table or a filter's survivors: launch latency is all
        dict(name="keys_5k", op="keys", n=5_000, dist="uniform"),
        # one frame's or one batch's records, where launches still dominate
        dict(name="pairs_60k", op="pairs", n=60_001, dist="uniform"),
        # the library's own small workload
        dict(name="keys_1m", op="keys", n=1 << 20, dist="uniform"),
        # an ordinary column argsort, a size no tile divides
        dict(name="pairs_10m", op="pairs", n=10_000_019, dist="uniform"),
        # low-entropy keys: flags, counters and small numbers beside large ones
        dict(name="pairs_64m_and4", op="pairs", n=1 << 26, dist="and4"),
        # the headline workload: key-value pairs at the largest size
        dict(name="pairs_256m", op="pairs", n=1 << 28, dist="uniform"),
        # the same size without values: building a sorted set
        dict(name="keys_256m", op="keys", n=1 << 28, dist="uniform"),
        # hashes or space-filling-curve codes of one scene with their indexes
        dict(name="pairs64_300k", op="pairs64", n=300_007, dist="uniform"),
        # the same for a large table
        dict(name="pairs64_64m", op="pairs64", n=1 << 26, dist="uniform"),
        # many uneven arrays in one call, up to 2^20 items each
        dict(name="batched_mix", op="batched", segments=4096, lo=6.0, hi=20.0, cap=1 << 27, sizes_seed=4,
             dist="uniform"),
        # many short rows in one call: adjacency lists, candidate lists
        dict(name="batched_rows", op="batched", segments=32768, lo=4.0, hi=11.0, cap=1 << 27, sizes_seed=9,
             dist="uniform"),
        # requests of mixed size and key distribution through the serving loop
        dict(name="serving_64", op="serving", requests=64, lo=10.0, hi=22.0, sizes_seed=5),
    ]


DISTS32 = ("uniform", "uniform", "uniform", "and2", "and4", "and8", "top_a5", "zipf16")
DISTS64 = ("uniform", "uniform", "uniform", "and2", "small", "low32")


def _log_size(rng, lo, hi):
    return int(2.0 ** rng.uniform(math.log2(lo), math.log2(hi)))


def draw(rng):
    op = rng.choice(("keys", "keys", "pairs", "pairs", "pairs", "keys64", "pairs64", "msd", "batched", "batched",
                     "serving"))
    if op in ("keys", "pairs"):
        return dict(op=op, n=_log_size(rng, 1 << 10, (1 << 28) * 0.9), dist=rng.choice(DISTS32))
    if op in ("keys64", "pairs64"):
        return dict(op=op, n=_log_size(rng, 1 << 10, 1 << 26), dist=rng.choice(DISTS64))
    if op == "msd":
        return dict(op=op, n=_log_size(rng, 1 << 18, (1 << 28) * 0.9), dist="uniform")
    if op == "batched":
        hi = rng.uniform(6.0, 20.0)
        lo = rng.uniform(4.0, hi - 1.0)
        # a total of 2^17 to 2^26 items, at most 2^16 segments
        mean = (2.0 ** hi - 2.0 ** lo) / ((hi - lo) * math.log(2.0))
        segments = int(min(1 << 16, max(2, _log_size(rng, 1 << 17, 1 << 26) / mean)))
        return dict(op=op, segments=segments, lo=lo, hi=hi, cap=1 << 26, sizes_seed=rng.randrange(1 << 30),
                    dist=rng.choice(("uniform", "uniform", "and4", "zipf16")))
    return dict(op=op, requests=rng.randint(4, 64), lo=10.0, hi=rng.uniform(12.0, 22.0),
                sizes_seed=rng.randrange(1 << 30))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _sizes(case):
    """Segment or request sizes, log-uniform; the same for every seed."""
    r = np.random.default_rng(case["sizes_seed"])
    if case["op"] == "serving":
        u = r.uniform(case["lo"], case["hi"], size=case["requests"])
        return np.floor(np.exp2(u)).astype(np.int64)
    u = r.uniform(case["lo"], case["hi"], size=case["segments"])
    sizes = np.floor(np.exp2(u)).astype(np.int64)
    if sizes.sum() > case["cap"]:
        sizes = np.maximum(1, sizes * case["cap"] // sizes.sum())
        sizes[int(np.argmax(sizes))] -= max(0, int(sizes.sum()) - case["cap"])
    return sizes


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _words32(n, g):
    return torch.randint(-(1 << 31), 1 << 31, (n,), dtype=torch.int32, device=DEV, generator=g)


def _words64(n, g):
    hi = torch.randint(-(1 << 31), 1 << 31, (n,), dtype=torch.int64, device=DEV, generator=g)
    return hi.bitwise_left_shift_(32).bitwise_or_(
        torch.randint(0, 1 << 32, (n,), dtype=torch.int64, device=DEV, generator=g))


def _keys32(dist, n, g):
    k = _words32(n, g)
    if dist.startswith("and"):
        for _ in range(int(dist[3:]) - 1):
            k.bitwise_and_(_words32(n, g))
    elif dist == "top_a5":  # 24 significant bits under a constant top byte
        k.bitwise_and_(0xFFFFFF).bitwise_or_((0xA5 << 24) - (1 << 32))
    elif dist == "zipf16":  # 16 distinct keys, rank frequencies r^-1.2
        dictionary = _words32(16, g)
        w = torch.arange(1, 17, dtype=torch.float64, device=DEV) ** -1.2
        edges = (torch.cumsum(w / w.sum(), 0)[:-1] * 2.0 ** 32 - 2.0 ** 31).to(torch.int32)
        k = dictionary[torch.bucketize(k, edges, out_int32=True)]
    return k


def _keys64(dist, n, g):
    k = _words64(n, g)
    if dist == "and2":
        k.bitwise_and_(_words64(n, g))
    elif dist == "small":  # below 2^20
        k.bitwise_and_((1 << 20) - 1)
    elif dist == "low32":  # 32-bit numbers in 64-bit keys
        k.bitwise_and_((1 << 32) - 1)
    return k


def _index(n):
    return torch.arange(n, dtype=torch.int32, device=DEV)


def _inputs(case, seed):
    """(keys, values or None) of a case with one array per pass."""
    g = _gen(seed)
    op = case["op"]
    if op == "batched":
        n = int(_sizes(case).sum())
        return _keys32(case["dist"], n, g), _index(n)
    n = case["n"]
    keys = _keys64(case["dist"], n, g) if op.endswith("64") else _keys32(case["dist"], n, g)
    return keys, _index(n) if op in ("pairs", "pairs64", "msd") else None


def _request_inputs(case, seed):
    """One (keys, values) pair per request."""
    g = _gen(seed)
    kinds = ("uniform", "and4", "zipf16")
    return [(_keys32(kinds[i % 3], int(n), g), _index(int(n))) for i, n in enumerate(_sizes(case))]


def prepare(case, seed):
    op = case["op"]
    state = {"op": op}
    if op == "serving":
        state["inputs"] = _request_inputs(case, seed)
        # the results of all requests side by side in one array each
        sizes = [int(n) for n in _sizes(case)]
        state["k"], state["v"] = (torch.empty(sum(sizes), dtype=torch.int32, device=DEV) for _ in range(2))
        state["outputs"] = list(zip(state["k"].split(sizes), state["v"].split(sizes)))
        state["server"] = rts.Server(hbm_budget_bytes=2 << 30, max_active=256)
        torch.cuda.synchronize()  # the server reads the inputs on a stream of its own
        return state
    keys, vals = _inputs(case, seed)
    state["keys"], state["vals"] = keys, vals
    state["k"] = torch.empty_like(keys)
    state["v"] = None if vals is None else torch.empty_like(vals)
    if op == "batched":
        off = np.zeros(case["segments"] + 1, dtype=np.int64)
        off[1:] = np.cumsum(_sizes(case))
        state["offsets"] = torch.from_numpy(off.astype(np.int32)).to(DEV)
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(state):
    op = state["op"]
    if op == "serving":
        server = state["server"]
        tickets = [server.submit(k, v, ok, ov) for (k, v), (ok, ov) in zip(state["inputs"], state["outputs"])]
        for t in tickets:
            server.wait(t)
        return state["k"], state["v"]
    k, v = state["k"], state["v"]
    k.copy_(state["keys"])
    if v is not None:
        v.copy_(state["vals"])
    if op == "keys":
        rts.sort_keys(k)
    elif op == "pairs":
        rts.sort_pairs(k, v)
    elif op == "keys64":
        rts.sort_keys64(k)
    elif op == "pairs64":
        rts.sort_pairs64(k, v)
    elif op == "msd":
        rts.sort_msd_first(k, v)
    else:
        rts.sort_pairs_batched(k, v, state["offsets"])
    return (k,) if v is None else (k, v)


def work(case):
    """Each key and value read once and written once; a sort computes nothing."""
    op = case["op"]
    n = int(_sizes(case).sum()) if op in ("batched", "serving") else case["n"]
    item = {"keys": 4, "keys64": 8, "pairs64": 12}.get(op, 8)
    return {"bytes": 2 * item * n, "flops": 0}


# ---------------------------------------------------------------------------
# the same outputs from torch
# ---------------------------------------------------------------------------

def _sorted32(keys, vals, segment=None):
    """A stable sort by unsigned key (inside each segment)."""
    order = keys.to(torch.int64).bitwise_and_((1 << 32) - 1)
    if segment is not None:
        order.bitwise_or_(segment.bitwise_left_shift(32))
    order, at = torch.sort(order, stable=True)
    out = order.bitwise_and_((1 << 32) - 1).to(torch.int32)
    return (out,) if vals is None else (out, vals[at])


def exact(case, seed):
    op = case["op"]
    if op == "serving":
        done = [_sorted32(k, v) for k, v in _request_inputs(case, seed)]
        return tuple(torch.cat(part) for part in zip(*done))
    keys, vals = _inputs(case, seed)
    if op == "batched":
        sizes = torch.from_numpy(_sizes(case)).to(DEV)
        segment = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), sizes)
        return _sorted32(keys, vals, segment)
    if not op.endswith("64"):
        return _sorted32(keys, vals)
    out, at = torch.sort(keys.bitwise_xor(SIGN64), stable=True)
    out.bitwise_xor_(SIGN64)
    return (out,) if vals is None else (out, vals[at])
