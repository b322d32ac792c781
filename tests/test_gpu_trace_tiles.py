"""Address digests (see test_gpu_trace.py) of what that file's workloads do not
reach: the tile sorts of 8192 and 16384 records, sorts of one routing pass (one
block, so its ticket is always the same), whose bins are compacted when the sort
is one tile and sorted otherwise, and the out-of-core calls.
"""
import numpy as np
import pytest

from gpu_util import trace_digests
from paper_2008_01765_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2008_01765_amd import bos  # noqa: E402

SLOTS = 1 << 21  # at least one per thread of the largest launch


@pytest.fixture(scope="module")
def digests():
    with trace_digests(SLOTS) as run:
        yield run


def _records(n, rec, data_seed):
    a = inputs.records(n, rec, data_seed)
    a[:, 0] >>= 1
    return a


def _sort(digests, a, **kw):
    st, route, sort = digests(bos.sort, bos.from_numpy(a), **kw)
    assert st == bos.OK
    return route, sort


@pytest.mark.parametrize("rec,tile", [(8, 8192), (8, 16384), (16, 8192)])
def test_big_tile_digests(digests, rec, tile):
    # one tile: its network is oblivious, so the whole sort is
    n = tile - 5
    a, b = _records(n, rec, 42), _records(n, rec, 43)
    ra, sa = _sort(digests, a, seed=1, z=512, tile=tile)
    rb, sb = _sort(digests, b, seed=1, z=512, tile=tile)
    assert torch.equal(ra, rb) and torch.equal(sa, sb)
    # the digest sees the tile's accesses: one record more is another digest
    _, sc = _sort(digests, _records(n + 1, rec, 42), seed=1, z=512, tile=tile)
    assert not torch.equal(sa, sc)


@pytest.mark.parametrize("rec,tile", [(8, 8192), (8, 16384), (16, 8192)])
def test_sorts_of_big_tiles_digests(digests, rec, tile):
    # more than 16 tiles: four-way passes over samples that the tiles wrote
    n = 20 * tile + 77
    a, b = _records(n, rec, 42), _records(n, rec, 43)
    c = a.copy()
    c[:, 0] = 2 * c[:, 0] + 1  # same order type
    (ra, sa), (rb, sb), (rc, sc) = [_sort(digests, x, seed=1, z=512, tile=tile) for x in (a, b, c)]
    assert torch.equal(ra, rb) and torch.equal(ra, rc)
    assert torch.equal(sa, sc)
    assert not torch.equal(sa, sb)


@pytest.mark.parametrize("rec", [8, 16])
@pytest.mark.parametrize("n,z,tile", [(1000, 512, 0), (1000, 512, 1024), (2000, 512, 1024), (2000, 1024, 0)])
def test_one_pass_digests(digests, rec, n, z, tile):
    a, b = _records(n, rec, 42), _records(n, rec, 43)
    ra, sa = _sort(digests, a, seed=1, z=z, tile=tile)
    rb, sb = _sort(digests, b, seed=1, z=z, tile=tile)
    assert int(torch.count_nonzero(ra)) > 0
    assert torch.equal(ra, rb)
    if n <= (tile or 4096):
        assert torch.equal(sa, sb)
    _, rc, _ = digests(bos.sort, bos.from_numpy(a), seed=2, z=z, tile=tile)
    assert not torch.equal(ra, rc)  # other labels, other loads


@pytest.mark.parametrize("fn", ["orp_host", "sort_host"])
def test_out_of_core_digests(digests, fn):
    # several trips of several chunks
    n = (1 << 19) + 4097
    got = []
    for data_seed in (42, 43):
        t = bos.pinned_empty((n, 2), torch.int32)
        t.numpy()[:] = _records(n, 8, data_seed).view(np.int32)
        st, route, sort = digests(getattr(bos, fn), t, seed=1, z=512, k=3)
        assert st == bos.OK
        got.append((route, sort))
    assert int(torch.count_nonzero(got[0][0])) > 0
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1]) == (fn == "orp_host")
