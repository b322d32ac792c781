"""Sorts whose plan is one routing pass: a sort of one tile only compacts its
bins in the fused last pass (the tile sort orders them), one of several tiles
sorts them.  Alone, batched and stepped; outputs are the records in (key, payload)
order.
"""
import numpy as np
import pytest

import closed_forms as cf
from paper_2008_01765_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2008_01765_amd import bos, serving  # noqa: E402


def _sizes(z, k):
    # one level up to the k levels of one pass, around the edges of their sizes
    return [n for n in (z // 2 + 1, z, z + 1, (z << k) // 2 - 1, (z << k) // 2) if n <= (z << k) // 2]


@pytest.mark.parametrize("rec", [8, 16])
@pytest.mark.parametrize("z,k,tile", [(16, 4, 4096), (32, 3, 4096), (256, 3, 4096), (256, 4, 1024), (512, 3, 4096),
                                      (512, 4, 1024), (1024, 2, 4096), (1024, 2, 1024), (2048, 1, 4096)])
def test_one_pass_plans(rec, z, k, tile):
    kw = {"z": z, "k": k, "tile": tile, "max_retries": 60, "min_security_bits": 0}
    # (the largest blocks of whole records do not fit a workgroup: two passes there)
    sizes = [n for n in _sizes(z, k)
             if len(bos.plan(n, rec, z=z, k=k, tile=tile, min_security_bits=0)["passes"]) == 1]
    assert sizes
    a = [inputs.records(n, rec, 90 + i, key_bits=6) for i, n in enumerate(sizes)]
    for x in a:
        out = bos.to_numpy(bos.sort(bos.from_numpy(x), seed=2, **kw))
        np.testing.assert_array_equal(out, cf.sorted_records(x))
    for x, o in zip(a, bos.sort_batched([bos.from_numpy(x) for x in a], list(range(len(a))), **kw)):
        np.testing.assert_array_equal(bos.to_numpy(o), cf.sorted_records(x))
    srv = serving.Server(hbm_budget_bytes=1 << 30, **kw)
    futs = [srv.submit(bos.from_numpy(x)) for x in a]
    srv.run_until_idle()
    for x, f in zip(a, futs):
        np.testing.assert_array_equal(bos.to_numpy(f.result()), cf.sorted_records(x))
