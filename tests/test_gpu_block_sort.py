"""The default sort of arrays that fit one block's LDS (bin sort, or digit
passes where keys crowd a bin), against the oracle, at the edges of its
shapes and of its range, over keys that take each method."""
import numpy as np
import pytest

import oracle
import paper_1008_2849_amd as rts
from paper_1008_2849_amd import inputs
from gpu_util import announce, sync, to_dev, to_host

pytestmark = pytest.mark.gpu


def keys32(kind, n, seed):
    u = inputs.uniform_keys(n, seed)
    if kind == "uniform":
        return u
    if kind == "one":  # a single value
        return np.full(n, 0x80000001, dtype=np.uint32)
    if kind == "ends":  # the two extreme keys only: two bins
        return np.where(u & 1, np.uint32(0xFFFFFFFF), np.uint32(0)).astype(np.uint32)
    if kind == "narrow":  # a range across a power of two, about four items a value
        return (np.uint32(0x7FFFFF00) + u % np.uint32(max(2, n // 4))).astype(np.uint32)
    if kind == "cluster":  # one far key widens the bins until they overflow
        u = u & np.uint32(0xFFFF)
        u[n // 2] = 0xFFFFFFFF
        return u
    return inputs.and_keys(n, 4, seed)


@pytest.mark.parametrize("kind", ["uniform", "one", "ends", "narrow", "cluster", "and4"])
@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 127, 128, 129, 257, 1023, 1024, 1025, 4096, 4097, 8191, 8193, 16383, 16384, 16385])
def test_small_sort(kind, n):
    announce(f"block sort {kind} n={n}")
    keys, vals = keys32(kind, n, 900 + n), inputs.index_values(n)
    rk, rv = oracle.lsd_sort(keys, vals)
    k, v, only = to_dev(keys), to_dev(vals), to_dev(keys)
    rts.sort_pairs(k, v)
    rts.sort_keys(only)
    sync()
    assert np.array_equal(to_host(k), rk) and np.array_equal(to_host(v), rv)
    assert np.array_equal(to_host(only), rk)


@pytest.mark.parametrize("kind", ["uniform", "small", "high", "low32", "and2"])
@pytest.mark.parametrize("n", [2, 65, 127, 128, 129, 1024, 1025, 4097, 8191, 8192, 8193])
def test_small_sort64(kind, n):
    import torch
    announce(f"block sort64 {kind} n={n}")
    keys = inputs.keys64(kind, n, 950 + n)
    order = np.argsort(keys, kind="stable")
    for vdt in (None, np.int32, np.int64):
        k = torch.from_numpy(keys.view(np.int64).copy()).cuda()
        v = None if vdt is None else torch.from_numpy(np.arange(n, dtype=vdt)).cuda()
        rts.sort64_ex(k, v)
        sync()
        assert np.array_equal(k.cpu().numpy().view(np.uint64), keys[order])
        if v is not None:
            assert np.array_equal(v.cpu().numpy(), order.astype(vdt))


def test_small_sort_leaves_its_neighbours():
    """A sort of a slice (4-byte aligned only) writes nothing around it, and a
    validated call with a workspace of its own reports success."""
    import torch
    n = 5001
    base = inputs.uniform_keys(n + 6, 77)
    for lo in (1, 2, 3):
        announce(f"block sort slice at {lo}")
        k = to_dev(base)
        cfg = rts.Config(flags=4)  # RT_FLAG_VALIDATE
        ws = torch.empty(rts.workspace_bytes(n, False, cfg), dtype=torch.uint8, device="cuda")
        rts.sort_ex(k[lo:lo + n], None, cfg, ws)
        sync()
        got = to_host(k)
        want = base.copy()
        want[lo:lo + n] = np.sort(base[lo:lo + n])
        assert np.array_equal(got, want)
