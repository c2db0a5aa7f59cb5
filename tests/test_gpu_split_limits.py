"""The limits of the splitter passes: malformed batched offsets whose
overlapping segments hold leaves that no LDS holds; the sizes on each side of
the lines where a method begins or ends."""
import numpy as np
import pytest

import paper_1008_2849_amd as rts
from paper_1008_2849_amd import inputs
from paper_1008_2849_amd._lib import RT_ERR_INVALID_ARG, RtError
from gpu_util import announce, sync, to_dev, to_host
from test_gpu_split import keys_of, sample_positions
from test_gpu_split_large import missed

pytestmark = pytest.mark.gpu


def miss_segment(keys, a, b, seed):
    """Moves the sampled keys of segment [a, b) out of the range of the rest."""
    at = a + np.unique(sample_positions(b - a, 2048))
    u = inputs.uniform_keys(len(at), seed)
    keys[at] = np.where(np.arange(len(at)) % 2 == 0, u % np.uint32(1 << 29), ~(u % np.uint32(1 << 29)))


def test_overlapping_long_leaves_stay_inside():
    """Offsets that decrease give two overlapping segments, each with a leaf
    sorted through global memory by its own block: the call reports them, what
    lies outside is not touched, and a well-formed segment behind is sorted."""
    ends = [1000, 91000, 31000, 121000, 171000]  # [91000, 31000) is malformed
    n, guard = ends[-1] + 1000, 50_000
    keys = inputs.uniform_keys(n, 5) % np.uint32(1 << 12) + np.uint32(1 << 30)
    for a, b in ((1000, 91000), (31000, 121000), (121000, 171000)):
        miss_segment(keys, a, b, a)
    vals = np.arange(n, dtype=np.uint32)
    edge = np.full(guard, 0xABCD1234, np.uint32)
    k, v = to_dev(np.concatenate([edge, keys, edge])), to_dev(np.concatenate([edge, vals, edge]))
    off = to_dev(np.array(ends, np.uint32) + np.uint32(guard))
    announce("batched, overlapping segments with long leaves")
    with pytest.raises(RtError) as e:
        rts.sort_batched_ex(k, v, off, 400_000, validate=True)
    assert e.value.status == RT_ERR_INVALID_ARG
    sync()
    gk, gv = to_host(k), to_host(v)
    for got, want in ((gk, keys), (gv, vals)):
        assert np.all(got[:guard] == edge) and np.all(got[-guard:] == edge)
        assert np.array_equal(got[guard:guard + 1000], want[:1000])
        assert np.array_equal(got[guard + 171000:guard + n], want[171000:])
    order = np.argsort(keys[121000:171000], kind="stable")
    assert np.array_equal(gk[guard + 121000:guard + 171000], keys[121000:171000][order])
    assert np.array_equal(gv[guard + 121000:guard + 171000], vals[121000:171000][order])


def leaf_ms(call):
    """Milliseconds that the call's leaf launches take, None if it has none."""
    rts.profile_start()
    call()
    sync()
    ms = [t for kind, t in rts.profile_stop() if kind == 8]
    return sum(ms) if ms else None


def words64(n, ands, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    k = torch.empty(n, dtype=torch.int64, device="cuda").random_(-(1 << 63), (1 << 63) - 1, generator=g)
    for _ in range(ands - 1):
        k &= torch.empty(n, dtype=torch.int64, device="cuda").random_(-(1 << 63), (1 << 63) - 1, generator=g)
    return k


def check_pairs64(k0, k, v):
    """The properties that fix a stable sort of original indices."""
    import torch
    n = k0.numel()
    s = k ^ (-(1 << 63))  # unsigned order as signed order
    assert bool((s[1:] >= s[:-1]).all()), "keys ascend"
    at = v.to(torch.int64)
    assert bool((torch.bincount(at, minlength=n) == 1).all()), "values are a permutation"
    assert bool(torch.equal(k0[at], k)), "each key arrives with its own index"
    eq = k[1:] == k[:-1]
    assert bool((at[1:][eq] > at[:-1][eq]).all()), "equal keys keep index order"


@pytest.mark.parametrize("ands", [1, 2])
@pytest.mark.parametrize("n,splitters", [(1 << 28, True), ((1 << 28) + 1, False)])
def test_where_two_passes_of_64_bit_keys_end(n, splitters, ands):
    """Two splitter passes up to 2^28 items, whose leaves the LDS holds; digit
    passes above."""
    import torch
    announce(f"64-bit keys, the end of two passes, n={n} ands={ands}")
    k0 = words64(n, ands, 7 + ands)
    k, v = k0.clone(), torch.arange(n, dtype=torch.int32, device="cuda")
    ms = leaf_ms(lambda: rts.sort_pairs64(k, v))
    assert ms > 0.5 if splitters else ms is None, ms
    check_pairs64(k0, k, v)
    del k0, k, v
    torch.cuda.empty_cache()


@pytest.mark.parametrize("kind,splitters", [("small", False), ("bytes", False), ("one", False), ("four bytes", True),
                                            ("outliers", True), ("uniform", True)])
def test_64_bit_keys_that_differ_in_few_bytes(kind, splitters):
    """From 2^27 items keys that differ in at most three bytes take digit
    passes, unless other keys are among them that the sample misses."""
    import torch
    n = 1 << 27
    announce(f"64-bit keys, {kind}, n={n}")
    k0 = words64(n, 1, 17)
    if kind == "bytes":
        k0 &= 0x7F0000FF0000FF00
    elif kind == "one":
        k0.fill_(-5)
    elif kind == "four bytes":
        k0 &= 0xFFFFFFFF
    elif kind != "uniform":
        k0 &= (1 << 20) - 1
    if kind == "outliers":
        k0[64 + 1000003::1000003] |= 0x0102030405060708
    k, v = k0.clone(), torch.arange(n, dtype=torch.int32, device="cuda")
    ms = leaf_ms(lambda: rts.sort64_ex(k, v))
    assert (ms > 0.3) == splitters, ms
    check_pairs64(k0, k, v)
    k.copy_(k0)
    rts.sort64_ex(k, None, rts.Config(flags=4))  # keys alone; waits, and reports what the kernels raised
    s = k ^ (-(1 << 63))
    assert bool((s[1:] >= s[:-1]).all()) and bool(torch.equal(k, k0[v.to(torch.int64)]))
    del k0, k, v, s
    torch.cuda.empty_cache()


M = 1 << 20  # the longest segment that takes a splitter pass


@pytest.mark.parametrize("kind", ["uniform", "and4", "zipf16", "one"])
@pytest.mark.parametrize("sizes", [[M], [M + 1], [M, M], [M + 1, M], [3 * M, M + 1], [M, 30_000, M + 1, 5, 16_385, M - 1],
                                   [2 * M + 7, 100, 20_000, 70_000]], ids=str)
def test_segments_around_the_longest_a_splitter_pass_takes(sizes, kind):
    announce(f"batched segments {sizes} {kind}")
    n = sum(sizes)
    keys = {"uniform": lambda: inputs.uniform_keys(n, 71), "and4": lambda: inputs.and_keys(n, 4, 72),
            "zipf16": lambda: inputs.zipf16_keys(n, 73), "one": lambda: np.full(n, 7, np.uint32)}[kind]()
    off = (np.concatenate([[0], np.cumsum(sizes)]) + 3).astype(np.uint32)
    base = np.concatenate([np.full(3, 9, np.uint32), keys, np.full(5, 9, np.uint32)])
    vals = np.arange(len(base), dtype=np.uint32)
    want_k, want_v = base.copy(), vals.copy()
    for a, b in zip(off[:-1], off[1:]):
        order = np.argsort(base[a:b], kind="stable")
        want_k[a:b], want_v[a:b] = base[a:b][order], vals[a:b][order]
    o, k, v, only = to_dev(off), to_dev(base), to_dev(vals), to_dev(base)
    rts.sort_batched_ex(k, v, o, n, validate=True)
    rts.sort_batched_ex(only, None, o, n, validate=True)
    sync()
    assert np.array_equal(to_host(k), want_k) and np.array_equal(to_host(v), want_v)
    assert np.array_equal(to_host(only), want_k)


@pytest.mark.parametrize("sizes", [
    [M + 1, 40, 300_000, 2 * M + 16_385, 17_000, 0, 64, 5 * M],           # too long by their mean
    [M + 1, 40, 300_000, 2 * M + 16_385, 17_000, 0, 64, 5 * M] + [9] * 4,  # most items too long
    [300_000] * 9 + [M + 1, 40, 17_000] + [260_000] * 9,                  # few of them
], ids=len)
def test_long_segments_of_two_streams_and_replays(sizes):
    """Segments above 2^20 items among shorter ones: two streams at once, each
    with a workspace of its own, then a captured call replayed on new keys."""
    import torch
    n = sum(sizes)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)
    o = to_dev(off)

    def expected(keys):
        order = np.concatenate([a + np.argsort(keys[a:b], kind="stable") for a, b in zip(off[:-1], off[1:])])
        return keys[order], order.astype(np.uint32)

    streams = [torch.cuda.Stream() for _ in range(2)]
    spaces = [torch.empty(rts.batched_workspace_bytes(len(sizes), n), dtype=torch.uint8, device="cuda") for _ in streams]
    inp = [inputs.uniform_keys(n, 81), inputs.and_keys(n, 4, 82)]
    want = [expected(x) for x in inp]
    k0, v0 = [to_dev(x) for x in inp], to_dev(inputs.index_values(n))
    k, v = [torch.empty_like(x) for x in k0], [torch.empty_like(v0) for _ in streams]
    announce("batched, segments above 2^20 items on two streams")
    sync()
    for rep in range(5):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                k[i].copy_(k0[i])
                v[i].copy_(v0)
                rts.sort_batched_ex(k[i], v[i], o, n, workspace=spaces[i], stream=s)
        sync()
        for i in range(2):
            assert np.array_equal(to_host(k[i]), want[i][0]) and np.array_equal(to_host(v[i]), want[i][1]), (rep, i)
    announce("the same, captured and replayed")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=streams[0]):
        rts.sort_batched_ex(k[0], v[0], o, n, workspace=spaces[0], stream=streams[0])
    for rep in range(4):
        k[0].copy_(k0[rep % 2])
        v[0].copy_(v0)
        sync()
        g.replay()
        sync()
        got = want[rep % 2]
        assert np.array_equal(to_host(k[0]), got[0]) and np.array_equal(to_host(v[0]), got[1]), rep


@pytest.mark.parametrize("sizes,splitters,digits", [
    ([20_000] * 52, True, False),                 # up to 2^20 items: no segment can be too long for a splitter pass
    ([20_000] * 53, False, True),                 # up to 2^22: one method's launches, not both's
    ([20_000] * 209, False, True),
    ([20_000] * 210, True, True),                 # above: splitters, and digit passes for what is too long
    ([2_000_000] * 3, False, True),               # too long by their mean
    ([5_000_000, 300_000, 20_000] + [64] * 4, True, True),     # most items too long: all by digit passes
    ([1_100_000] + [130_000] * 40 + [64] * 4, True, True),     # few of them
], ids=lambda x: f"{len(x)}x{x[0]}" if isinstance(x, list) else None)
def test_method_of_a_batched_call(sizes, splitters, digits):
    announce(f"method of {len(sizes)} segments of {sizes[0]}")
    n = sum(sizes)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)
    keys = inputs.and_keys(n, 2, 91)
    order = np.concatenate([a + np.argsort(keys[a:b], kind="stable") for a, b in zip(off[:-1], off[1:])])
    k, v, o = to_dev(keys), to_dev(inputs.index_values(n)), to_dev(off)
    rts.profile_start()
    rts.sort_batched_ex(k, v, o, n)
    sync()
    kinds = {kind for kind, _ in rts.profile_stop()}
    assert (10 in kinds) == splitters and (17 in kinds) == digits, kinds
    assert np.array_equal(to_host(k), keys[order]) and np.array_equal(to_host(v), order.astype(np.uint32))


def timed(call):
    """Milliseconds of a call, the second of two."""
    import torch
    for _ in range(2):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        sync()
    return a.elapsed_time(b)


@pytest.mark.parametrize("with_values", [True, False])
@pytest.mark.parametrize("n", [(1 << 18) + 5, 1 << 20])
def test_keys_the_sample_misses(n, with_values):
    """Nearly all keys in one bucket, which the whole grid sorts: the result,
    and a time that one block alone does not reach (9 ms at 2^20)."""
    import torch
    announce(f"missed by the sample, n={n} values={with_values}")
    keys, vals = keys_of("missed", n, 31, np.uint32), inputs.index_values(n)
    order = np.argsort(keys, kind="stable")
    k0, v0 = to_dev(keys), to_dev(vals)
    k, v = torch.empty_like(k0), torch.empty_like(v0) if with_values else None

    def call():
        k.copy_(k0)
        if with_values:
            v.copy_(v0)
        rts.sort_ex(k, v, rts.Config(flags=4))
    ms = timed(call)
    assert np.array_equal(to_host(k), keys[order])
    assert not with_values or np.array_equal(to_host(v), order.astype(np.uint32))
    print(f"{ms:.3f} ms", flush=True)
    assert ms < 4.0


@pytest.mark.parametrize("vdt", [None, np.int32, np.int64])
def test_64_bit_keys_both_samples_miss(vdt):
    import torch
    n = (1 << 22) + 11
    announce(f"64-bit keys missed by both samples, n={n} values={vdt}")
    keys = missed(n, 3, 2048, True)
    order = np.argsort(keys, kind="stable")
    k0 = torch.from_numpy(keys.view(np.int64).copy()).cuda()
    k, v = torch.empty_like(k0), None
    if vdt is not None:
        v0 = torch.arange(n, device="cuda").to(torch.int32 if vdt == np.int32 else torch.int64)
        v = torch.empty_like(v0)

    def call():
        k.copy_(k0)
        if v is not None:
            v.copy_(v0)
        rts.sort64_ex(k, v, rts.Config(flags=4))
    ms = timed(call)
    assert np.array_equal(k.cpu().numpy().view(np.uint64), keys[order])
    assert v is None or np.array_equal(v.cpu().numpy(), order.astype(vdt))
    print(f"{ms:.3f} ms", flush=True)
    assert ms < 20.0  # one block alone: 77 ms


def test_keys_that_samples_miss_on_two_streams():
    """Two sorts whose leaves take the whole grid, at once: each goes on with
    whatever blocks of it are on the chip."""
    import torch
    a, b = keys_of("missed", 1 << 20, 33, np.uint32), missed((1 << 22) + 11, 5, 2048, True)
    ka, kb = to_dev(a), torch.from_numpy(b.view(np.int64).copy()).cuda()
    streams = [torch.cuda.Stream() for _ in range(2)]
    x, y = [torch.empty_like(ka) for _ in range(4)], torch.empty_like(kb)
    announce("two sorts of missed keys at once")
    sync()
    for rep in range(3):
        with torch.cuda.stream(streams[0]):
            for k in x:
                k.copy_(ka)
                rts.sort_keys(k, stream=streams[0])
        with torch.cuda.stream(streams[1]):
            y.copy_(kb)
            rts.sort_keys64(y, stream=streams[1])
        sync()
        assert all(np.array_equal(to_host(k), np.sort(a)) for k in x), rep
        assert np.array_equal(y.cpu().numpy().view(np.uint64), np.sort(b)), rep


@pytest.mark.parametrize("own,digits", [(None, True), (50_000, True), (1 << 20, False)])
def test_tuning_table_entry_of_a_small_size(own, digits, tmp_path):
    """A loaded table's entry sets the digit passes of default calls, unless the
    table leaves that size to the library's own methods."""
    import json
    n = 100_003
    announce(f"tuned shape at n={n}, own methods up to {own}")
    table = {"entries": [{"op": "pairs", "min_n": 0, "max_n": 1 << 20, "digit_bits": [8, 8, 8, 8], "block": 512,
                          "ipt": 16, "flags": 0}]}
    if own is not None:
        table["own_methods_max_n"] = own
    path = tmp_path / "t.json"
    path.write_text(json.dumps(table))
    keys, vals = inputs.uniform_keys(n, 19), inputs.index_values(n)
    order = np.argsort(keys, kind="stable")
    try:
        rts.load_tuning(str(path))
        for with_values, by_digits in ((True, digits), (False, False)):  # (no entry for keys alone)
            k, v = to_dev(keys), to_dev(vals)
            rts.profile_start()
            rts.sort_ex(k, v if with_values else None)
            sync()
            kinds = {kind for kind, _ in rts.profile_stop()}
            assert (19 in kinds) == by_digits and (8 in kinds) != by_digits, kinds
            assert np.array_equal(to_host(k), keys[order])
            assert not with_values or np.array_equal(to_host(v), order.astype(np.uint32))
    finally:
        rts.load_default_tuning()
