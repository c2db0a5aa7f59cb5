"""Arrays above 2^20 items (32-bit keys) and 2^19 items (64-bit keys, which take
one splitter pass up to 600064 items and two from 2^22) against a stable host
sort: tile and leaf edges, repeated keys (long buckets of one value), and keys
that the passes' samples miss (a leaf no LDS holds)."""
import numpy as np
import pytest

import paper_1008_2849_amd as rts
from paper_1008_2849_amd import inputs
from gpu_util import announce, sync
from test_gpu_split import keys_of, sample_positions

pytestmark = pytest.mark.gpu


def missed(n, seed, m, twice):
    """Nearly all keys in [2^30, 2^30 + 2^12), a range that none of the m keys
    sampled first falls in, nor (twice) those of the second pass, whose sample
    is of the one bucket those keys make."""
    u = inputs.uniform_keys(n, seed).astype(np.uint64)
    top = np.uint64((1 << 64) - 1)
    span = np.uint64(1 << 28)
    k = u % np.uint64(1 << 12) + np.uint64(1 << 30)
    at = sample_positions(n, m)
    k[at] = np.where(np.arange(m) % 2 == 0, u[at] % span, top - u[at] % span)
    if not twice:
        return k
    # the bucket those keys fall in, in input order: between two neighbours of
    # the sample's every (m / 256)-th key
    ordered = np.sort(k[at])
    rest = np.nonzero((k >= ordered[m // 2 - 1]) & (k < ordered[m // 2 + m // 256 - 1]))[0]
    again = rest[np.unique(sample_positions(len(rest), 2048))]
    low = np.arange(len(again)) % 2 == 0
    k[again] = np.where(low, np.uint64(1 << 29) + u[again] % span, np.uint64(1 << 31) - u[again] % span)
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
    announce(f"large {kind} n={n}")
    keys = keys_of(kind, n, 40 + n % 13, np.uint32)
    check(keys, None)
    check(keys, np.int32)


@pytest.mark.parametrize("kind", ["uniform", "zipf16", "extremes", "one", "and4"])
@pytest.mark.parametrize("n", [(1 << 19) + 1, 600_064, 600_065, 3_000_017, 1 << 22, 5_000_011])
def test_large64(kind, n):
    announce(f"large64 {kind} n={n}")
    keys = keys_of(kind, n, 50 + n % 13, np.uint64)
    for vdt in (None, np.int32, np.int64):
        check(keys, vdt)


@pytest.mark.parametrize("n", [590_001, 2_000_003, (1 << 22) + 3])
@pytest.mark.parametrize("kind", ["small", "high", "low32"])
def test_large64_in_some_bytes(kind, n):
    announce(f"large64 {kind} n={n}")
    check(inputs.keys64(kind, n, 5), np.int32)


@pytest.mark.parametrize("n,m,twice", [((1 << 19) + 4099, 8192, False), ((1 << 22) + 4099, 2048, True)])
def test_large_with_a_leaf_no_lds_holds(n, m, twice):
    announce(f"large64, the samples miss, n={n}")
    check(missed(n, 3, m, twice), np.int32)
    check(missed(n, 3, m, twice), None)
