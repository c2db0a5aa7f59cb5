"""The splitter sort (arrays above one block's LDS, up to 2^20 items with
32-bit keys and 2^19 with 64-bit keys) against the oracle: the edges of its
tile and leaf sizes, repeated keys (buckets of one value, longer than a leaf),
and keys chosen so that the sample misses nearly all of them (a bucket no leaf
holds)."""
import numpy as np
import pytest

import oracle
import paper_1008_2849_amd as rts
from paper_1008_2849_amd import inputs
from gpu_util import announce, sync, to_dev, to_host

pytestmark = pytest.mark.gpu


def sample_positions(n, m):
    """Where the kernel samples: a hashed item of each of m equal stretches."""
    i = np.arange(m, dtype=np.uint64)
    a, b = i * np.uint64(n) // np.uint64(m), (i + np.uint64(1)) * np.uint64(n) // np.uint64(m)
    h = ((i + np.uint64(1)) * np.uint64(0x9E3779B9)) & np.uint64(0xFFFFFFFF)
    return (a + ((h * (b - a)) >> np.uint64(32))).astype(np.int64)


def keys_of(kind, n, seed, dtype):
    u = inputs.uniform_keys(n, seed) if dtype == np.uint32 else inputs.uniform_keys64(n, seed)
    top = dtype(np.iinfo(dtype).max)
    if kind == "uniform":
        return u
    if kind == "sorted":
        return np.sort(u)
    if kind == "zipf16":
        return inputs.zipf16_keys(n, seed).astype(dtype) << dtype(8 * (np.dtype(dtype).itemsize - 4))
    if kind == "extremes":  # the smallest and the largest key, and one between
        return np.where(u % 3 == 0, dtype(0), np.where(u % 3 == 1, top, top - dtype(1))).astype(dtype)
    if kind == "one":
        return np.full(n, 0x80000001, dtype=dtype)
    if kind == "and4":
        return u & np.roll(u, 1) & np.roll(u, 2) & np.roll(u, 3)
    # "missed": what is not sampled lies in a range that holds no sample key
    k = (u % dtype(1 << 20)) + dtype(1 << 30)
    m = 4096 if n > 1 << 18 else 2048
    at = sample_positions(n, m)
    k[at] = np.where(np.arange(m) % 2 == 0, u[at] % dtype(1 << 29), (u[at] % dtype(1 << 29)) + (top - dtype(1 << 29)))
    return k


@pytest.mark.parametrize("kind", ["uniform", "sorted", "zipf16", "extremes", "one", "and4", "missed"])
@pytest.mark.parametrize("n", [16385, 20001, 65536, 65537, 131072, 131073, 262145, 524289, 1 << 20])
def test_split_sort(kind, n):
    if kind == "missed" and n > 262145:
        n = 262145 + n % 7  # the fallback runs on one block: a small one shows it
    announce(f"split sort {kind} n={n}")
    keys, vals = keys_of(kind, n, 700 + n % 97, np.uint32), inputs.index_values(n)
    rk, rv = oracle.lsd_sort(keys, vals)
    k, v, only = to_dev(keys), to_dev(vals), to_dev(keys)
    rts.sort_pairs(k, v)
    rts.sort_keys(only)
    sync()
    assert np.array_equal(to_host(k), rk) and np.array_equal(to_host(v), rv)
    assert np.array_equal(to_host(only), rk)


@pytest.mark.parametrize("kind", ["uniform", "zipf16", "extremes", "and4", "missed"])
@pytest.mark.parametrize("n", [8193, 65537, 131073, 262145, 1 << 19])
def test_split_sort64(kind, n):
    import torch
    if kind == "missed" and n > 131073:
        n = 131073 + n % 7
    announce(f"split sort64 {kind} n={n}")
    keys = keys_of(kind, n, 800 + n % 97, np.uint64)
    order = np.argsort(keys, kind="stable")
    for vdt in (None, np.int32, np.int64):
        k = torch.from_numpy(keys.view(np.int64).copy()).cuda()
        v = None if vdt is None else torch.from_numpy(np.arange(n, dtype=vdt)).cuda()
        rts.sort64_ex(k, v)
        sync()
        assert np.array_equal(k.cpu().numpy().view(np.uint64), keys[order])
        if v is not None:
            assert np.array_equal(v.cpu().numpy(), order.astype(vdt))


def test_split_sort_in_a_workspace_and_a_graph():
    """With a caller's workspace the call only launches kernels: a captured
    graph, replayed on new keys of a slice, gives each time the eager result."""
    import torch
    n = 100_003
    ws = torch.empty(rts.workspace_bytes(n, True), dtype=torch.uint8, device="cuda")
    k, v = to_dev(np.zeros(n + 4, np.uint32)), to_dev(np.zeros(n + 4, np.uint32))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            rts.sort_ex(k[3:n + 3], v[3:n + 3], None, ws, stream=s)
    torch.cuda.current_stream().wait_stream(s)
    for r in range(4):
        announce(f"split sort graph replay {r}")
        base = inputs.uniform_keys(n + 4, 60 + r) if r != 2 else keys_of("and4", n + 4, 62, np.uint32)
        k.copy_(to_dev(base))
        v.copy_(to_dev(inputs.index_values(n + 4)))
        g.replay()
        sync()
        order = np.argsort(base[3:n + 3], kind="stable")
        got, gv = to_host(k), to_host(v)
        assert np.array_equal(got[3:n + 3], base[3:n + 3][order])
        assert np.array_equal(gv[3:n + 3], (order + 3).astype(np.uint32))
        assert np.array_equal(got[:3], base[:3]) and got[n + 3] == base[n + 3]
