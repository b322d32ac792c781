"""An attempt that overflows is abandoned before anything orders its records.

The comparison sort's addresses depend on the order of the records it is given;
Section 3.3 allows that for a permuted array, which an aborted attempt is not.
With the digest build (see test_gpu_trace.py) a call whose only attempt overflows
must leave equal digests for two different inputs, in the comparison sort's
buffer too.
"""
import numpy as np
import pytest

import closed_forms as cf
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


# one rank launch (16 tiles), two- and four-way passes from narrow and wide tiles
@pytest.mark.parametrize("rec", [8, 16])
@pytest.mark.parametrize("n,tile", [((1 << 14) - 5, 1024), (1 << 16, 1024), ((1 << 17) - 77, 4096),
                                    ((1 << 19) - 1, 2048), ((1 << 19) - 1, 8192)])
@pytest.mark.parametrize("sync", [True, False])
def test_overflowed_sort_orders_nothing(digests, rec, n, tile, sync):
    # attempt 0 of this seed overflows at Z = 32
    kw = dict(seed=5, z=32, tile=tile, max_retries=0, min_security_bits=0)
    got = []
    for data_seed in (42, 43):
        t = bos.from_numpy(inputs.records(n, rec, data_seed))
        st, route, sort = digests(bos.sort, t, sync=sync, out=torch.empty_like(t), **kw)
        if sync:
            assert st == bos.OVERFLOW
        else:
            assert st == bos.OK and bos.status_word(t, z=32, tile=tile, min_security_bits=0) is not None
        got.append((route, sort))
    assert int(torch.count_nonzero(got[0][0])) > 0
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])


def _host(n, data_seed):
    a = inputs.records(n, 8, data_seed)
    t = bos.pinned_empty((n, 2), torch.int32)
    t.numpy()[:] = a.view(np.int32)
    return a, t


# Out of core, four chunks in the last trip: the loads of its levels counted ahead
# (k = 3), or too many of them and the runs sorted apart (k = 7).  Attempt 0 of these
# seeds overflows once, in the trip's third chunk (313) or second (431).
@pytest.mark.parametrize("k", [3, 7])
@pytest.mark.parametrize("seed", [313, 431])
def test_overflow_in_a_late_chunk_orders_nothing(digests, seed, k):
    n, z = 1 << 19, 64
    got = []
    for data_seed in (42, 43):
        _, t = _host(n, data_seed)
        st, route, sort = digests(bos.sort_host, t, seed=seed, z=z, k=k, max_retries=0, min_security_bits=0)
        assert st == bos.OVERFLOW
        got.append((route, sort))
    assert int(torch.count_nonzero(got[0][0])) > 0
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])


# seeds whose attempt 0 overflows in the first trip (109), in the last one (99, 313,
# 431) or not at all
@pytest.mark.parametrize("k", [3, 7])
@pytest.mark.parametrize("seed", [99, 109, 313, 314, 431, 432])
def test_overflow_found_out_of_core(seed, k):
    n, z, L = 1 << 19, 64, 14
    a, t = _host(n, 42)
    want = cf.first_overflow(n, cf.labels(seed, 0, n, L), 1 << L, L, z)
    got, rep = bos.sort_host(t, seed=seed, z=z, k=k, min_security_bits=0, report=True)
    assert (rep["first_overflow_level"], rep["first_overflow_pair"]) == want
    assert rep["attempts"] == (1 if want[0] < 0 else 2)
    np.testing.assert_array_equal(got.numpy().view(np.uint32), cf.sorted_records(a))


def test_retry_after_an_abandoned_attempt():
    # the next attempt's comparison sort runs
    a = inputs.records(1 << 14, 8, 42)
    want = cf.sorted_records(a)
    retried = 0
    for seed in range(11, 17):
        got, rep = bos.sort(bos.from_numpy(a), seed=seed, z=32, max_retries=30, min_security_bits=0, report=True)
        retried += rep["attempts"] > 1
        np.testing.assert_array_equal(bos.to_numpy(got), want)
    assert retried > 0
