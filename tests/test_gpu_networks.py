"""Edges of the routing and finish networks (bucket ORP, Sections 3.1 and 3.2).

* Labels longer than the count field of the marks prefix: at Z = 2048 a label
  of 20 bits or more takes the cut before the count (n > 2^29 there).
* Groups whose first element is not a multiple of 8 (the labels come in
  Philox blocks of 8), and groups of few elements: outputs against the oracle
  and the closed form over every Z.
"""
import numpy as np
import pytest

from gpu_util import torch_is_sorted

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2008_01765_amd import bos, inputs  # noqa: E402


@pytest.fixture(scope="module")
def ora():
    import oracle
    oracle.build(force=False)
    return oracle


def test_labels_longer_than_the_count_field():
    n = (1 << 29) + 1
    x = torch.empty((n, 2), dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x[:, 0] = torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, dtype=torch.int32, device="cuda")
    x[:, 1] = torch.arange(n, dtype=torch.int32, device="cuda")
    assert bos.plan(n, 8, z=2048)["levels"] == 20
    out = bos.sort(x, seed=3, z=2048)
    assert torch_is_sorted(out)
    # every record once: payloads are a permutation and carry their keys
    p = out[:, 1].to(torch.int64)
    seen = torch.zeros(n, dtype=torch.bool, device="cuda")
    seen[p] = True
    assert bool(seen.all())
    assert torch.equal(x[p, 0], out[:, 0])
    del x, out, p, seen
    bos.release_workspaces()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("rec", [8, 16])
@pytest.mark.parametrize("z", [16, 32, 64, 128, 256, 512, 1024, 2048])
@pytest.mark.parametrize("groups", ["full", "full_less_one", "half_more_one"])
def test_group_starts_of_every_alignment(ora, rec, z, groups):
    # n = B Z / 2 (aligned, full groups), one less (every start unaligned, some
    # groups a whole Z/2), and just over half of it (the smallest groups of a plan)
    b = 64
    n = {"full": b * z // 2, "full_less_one": b * z // 2 - 1, "half_more_one": b * z // 4 + 1}[groups]
    a = inputs.records(n, rec, 17)
    for attempt_seed in (1, 2):
        got = bos.to_numpy(bos.orp(bos.from_numpy(a), seed=attempt_seed, z=z, min_security_bits=0, max_retries=40))
        want = ora.orp(a, attempt_seed, z=z, max_retries=40)
        assert want["rc"] == 0
        np.testing.assert_array_equal(got, want["out"])
