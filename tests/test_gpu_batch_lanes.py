"""Batched routing launches with and without lane guards: blocks of at least
1024 slots fill their waves and run the unguarded kernels, smaller ones (Z = 256
at one and two levels per pass, Z = 32) the guarded ones.  Every instance comes
out in (key, payload) order.
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
@pytest.mark.parametrize("z,k", [(32, 2), (256, 1), (256, 2), (256, 3), (512, 1), (512, 2), (512, 4), (1024, 1),
                                 (1024, 2)])
def test_batch_of_every_block_size(rec, z, k):
    sizes = [1, 2 * z, 3 * z + 1, 16 * z - 3, 40 * z + 7]
    a = [inputs.records(n, rec, 80 + i) for i, n in enumerate(sizes)]
    outs = bos.sort_batched([bos.from_numpy(x) for x in a], list(range(len(sizes))), z=z, k=k, max_retries=60,
                            min_security_bits=0)
    for x, o in zip(a, outs):
        np.testing.assert_array_equal(bos.to_numpy(o), cf.sorted_records(x))
