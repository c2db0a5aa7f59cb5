"""The limits of the splitter passes: malformed batched offsets whose
overlapping segments hold leaves that no LDS holds."""
import numpy as np
import pytest

import paper_1008_2849_amd as rts
from paper_1008_2849_amd import inputs
from paper_1008_2849_amd._lib import RT_ERR_INVALID_ARG, RtError
from gpu_util import announce, sync, to_dev, to_host
from test_gpu_split import sample_positions

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
