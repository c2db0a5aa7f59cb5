"""The two-pass splitter sort (arrays above 2^20 items with 32-bit keys, 2^19
with 64-bit keys) against a stable host sort: tile and leaf edges, repeated
keys (long buckets of one value), and keys that both passes' samples miss (a
leaf no LDS holds)."""
import numpy as np
import pytest

import paper_1008_2849_amd as rts
from paper_1008_2849_amd import inputs
from gpu_util import announce, sync
from test_gpu_split import keys_of, sample_positions

pytestmark = pytest.mark.gpu


def missed_twice(n, seed, dtype):
    """Nearly all keys in [2^30, 2^30 + 2^12), a range that no sampled key of
    the first pass falls in, nor of the second, whose sample is of the one
    bucket those keys make."""
    m = 8192
    u = inputs.uniform_keys(n, seed).astype(dtype)
    top = dtype(np.iinfo(dtype).max)
    k = u % dtype(1 << 12) + dtype(1 << 30)
    at = sample_positions(n, m)
    k[at] = np.where(np.arange(m) % 2 == 0, u[at] % dtype(1 << 28), top - u[at] % dtype(1 << 28))
    # the bucket those keys fall in, in input order: between two neighbours of
    # the sample's every (m / 256)-th key
    ordered = np.sort(k[at])
    rest = np.nonzero((k >= ordered[m // 2 - 1]) & (k < ordered[m // 2 + m // 256 - 1]))[0]
    again = rest[np.unique(sample_positions(len(rest), 2048 if len(rest) < 1 << 19 else 4096))]
    low = np.arange(len(again)) % 2 == 0
    k[again] = np.where(low, dtype(1 << 29) + u[again] % dtype(1 << 28), dtype(1 << 31) - u[again] % dtype(1 << 28))
    return k


def check(keys, vdt, **kw):
    import torch
    kt = np.int32 if keys.dtype == np.uint32 else np.int64
    order = np.argsort(keys, kind="stable")
    k = torch.from_numpy(keys.view(kt).copy()).cuda()
    v = None if vdt is None else torch.from_numpy(np.arange(len(keys), dtype=vdt)).cuda()
    if keys.dtype == np.uint32:
        rts.sort_ex(k, v, rts.Config(flags=4), **kw)
    else:
        rts.sort64_ex(k, v, rts.Config(flags=4), **kw)
    sync()
    assert np.array_equal(k.cpu().numpy().view(keys.dtype), keys[order])
    if v is not None:
        assert np.array_equal(v.cpu().numpy(), order.astype(vdt))


@pytest.mark.parametrize("kind", ["uniform", "sorted", "zipf16", "extremes", "one", "and4"])
@pytest.mark.parametrize("n", [(1 << 20) + 1, 1_600_003, 1 << 22, 10_000_019])
def test_large32(kind, n):
    announce(f"two-pass split {kind} n={n}")
    keys = keys_of(kind, n, 40 + n % 13, np.uint32)
    check(keys, None)
    check(keys, np.int32)


@pytest.mark.parametrize("kind", ["uniform", "zipf16", "extremes", "one", "and4"])
@pytest.mark.parametrize("n", [(1 << 19) + 1, 3_000_017])
def test_large64(kind, n):
    announce(f"two-pass split64 {kind} n={n}")
    keys = keys_of(kind, n, 50 + n % 13, np.uint64)
    for vdt in (None, np.int32, np.int64):
        check(keys, vdt)


@pytest.mark.parametrize("kind", ["small", "high", "low32"])
def test_large64_in_some_bytes(kind):
    announce(f"two-pass split64 {kind}")
    check(inputs.keys64(kind, 2_000_003, 5), np.int32)


def test_large_with_a_leaf_no_lds_holds():
    n = (1 << 20) + 4099
    announce("two-pass split, both samples miss")
    check(missed_twice(n, 3, np.uint32), np.int32)
    check(missed_twice(n, 3, np.uint32), None)
    check(missed_twice(600_011, 4, np.uint64), np.int64)


def test_large_slices_and_a_workspace():
    import torch
    n = 1_500_001
    announce("two-pass split of a slice in a caller's workspace")
    base = inputs.uniform_keys(n + 2, 9)
    k = torch.from_numpy(base.view(np.int32).copy()).cuda()
    v = torch.arange(n + 2, dtype=torch.int32, device="cuda")
    ws = torch.empty(rts.workspace_bytes(n, True), dtype=torch.uint8, device="cuda")
    rts.sort_ex(k[1:n + 1], v[1:n + 1], None, ws)
    sync()
    order = np.argsort(base[1:n + 1], kind="stable") + 1
    got, gv = k.cpu().numpy().view(np.uint32), v.cpu().numpy()
    assert np.array_equal(got[1:n + 1], base[order]) and np.array_equal(gv[1:n + 1], order)
    assert got[0] == base[0] and got[n + 1] == base[n + 1] and gv[0] == 0 and gv[n + 1] == n + 1
