"""Trips of the out-of-core calls (Section 4.3): a chunk runs several routing
passes on the device before it leaves, and the sort's last trip strips and sorts
its chunks there.

Device workspaces from the smallest one up, so that the same plan takes several
trips (segments of 2^K buckets apart), two, and one chunk in all; outputs must
equal the in-core permutation and the records in (key, payload) order.
"""
import ctypes as C

import numpy as np
import pytest

import closed_forms as cf
from paper_2008_01765_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2008_01765_amd import bos  # noqa: E402


def _host(a):
    t = bos.pinned_empty(a.shape, torch.int32 if a.dtype == np.uint32 else torch.int64)
    t.numpy()[:] = a.view(np.int32 if a.dtype == np.uint32 else np.int64)
    return t


def _np(t, rec):
    return t.numpy().view(np.uint32 if rec == 8 else np.uint64)


def _device_bytes(n, rec, z, k):
    p = bos.params(0, z, k, 0)
    return bos.lib().bos_host_device_bytes(n, rec, C.byref(p))


@pytest.mark.parametrize("rec", [8, 16])
@pytest.mark.parametrize("z,k", [(512, 1), (512, 3), (512, 4), (256, 4), (1024, 2), (2048, 1)])
@pytest.mark.parametrize("times", [1, 3, 40])
def test_trips(rec, z, k, times):
    n = (1 << 20) + 4097 if rec == 8 else (1 << 19) + 4099
    a = inputs.records(n, rec, 71, key_bits=(18 if rec == 16 else None))
    ws = times * _device_bytes(n, rec, z, k)
    got = _np(bos.orp_host(_host(a), seed=5, z=z, k=k, dev_ws_bytes=ws, min_security_bits=0), rec)
    want = bos.to_numpy(bos.orp(bos.from_numpy(a), seed=5, z=z, k=k, min_security_bits=0))
    np.testing.assert_array_equal(got, want)
    got = _np(bos.sort_host(_host(a), seed=5, z=z, k=k, dev_ws_bytes=ws, min_security_bits=0), rec)
    np.testing.assert_array_equal(got, cf.sorted_records(a))


def test_tags_of_two_bytes():
    # 17 levels at the smallest workspace: trips of 8, 3, 3 and 3 levels, so the
    # slots cross the link with 9, 6 and 3 label bits left (tags of 2, 1 and 1 bytes)
    n = (1 << 24) + 1
    a = inputs.records(n, 8, 73)
    got = _np(bos.orp_host(_host(a), seed=6, z=512, k=3), 8)
    np.testing.assert_array_equal(got, bos.to_numpy(bos.orp(bos.from_numpy(a), seed=6, z=512)))
    got = _np(bos.sort_host(_host(a), seed=6, z=512, k=3), 8)
    np.testing.assert_array_equal(got, cf.sorted_records(a))


def test_sort_overflow_retries():
    # Z = 32 overflows often at this size: the overflowed attempts form no runs
    n = 1 << 14
    a = inputs.records(n, 8, 72)
    retried = 0
    for seed in range(11, 17):
        got, rep = bos.sort_host(_host(a), seed=seed, z=32, max_retries=30, min_security_bits=0, report=True)
        _, wrep = bos.orp(bos.from_numpy(a), seed=seed, z=32, max_retries=30, min_security_bits=0, report=True)
        assert rep["attempts"] == wrep["attempts"]
        retried += rep["attempts"] > 1
        np.testing.assert_array_equal(_np(got, 8), cf.sorted_records(a))
    assert retried > 0
