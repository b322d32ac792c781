"""One-launch merge of a small sort (at most 16 tiles): every record's rank is
its index in its run plus the records before it in the other runs.

Sizes at the edges of the path (two runs with one record in the second, 16
full runs, a ragged last run, one run more than it takes) and repeated records,
whose windows exceed the LDS ones and whose ties cross every run; single-tile
sorts at the edges of the smaller networks.  Expected: the records in
(key, payload) order.
"""
import numpy as np
import pytest

import closed_forms as cf
from paper_2008_01765_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2008_01765_amd import bos  # noqa: E402


@pytest.mark.parametrize("rec", [8, 16])
@pytest.mark.parametrize("tile,runs,extra", [(1024, 1, 1), (1024, 15, 257), (1024, 16, 0), (1024, 16, 1),
                                             (4096, 2, -1), (4096, 7, 255), (4096, 16, 0), (4096, 16, -1)])
@pytest.mark.parametrize("distinct", [0, 1, 5])
def test_one_pass_merge(rec, tile, runs, extra, distinct):
    n = tile * runs + extra
    a = inputs.records(n, rec, 23)
    if distinct:  # whole records repeated
        a = a[np.random.default_rng(distinct).integers(0, distinct, n)]
    out = bos.to_numpy(bos.sort(bos.from_numpy(a), seed=3, tile=tile, min_security_bits=0))
    np.testing.assert_array_equal(out, cf.sorted_records(a))


@pytest.mark.parametrize("rec", [8, 16])
@pytest.mark.parametrize("n", [2, 1023, 1024, 1025, 2048, 2049, 4096])
def test_single_tile_networks(rec, n):
    a = inputs.records(n, rec, 29)
    out = bos.to_numpy(bos.sort(bos.from_numpy(a), seed=3, tile=4096, min_security_bits=0))
    np.testing.assert_array_equal(out, cf.sorted_records(a))
