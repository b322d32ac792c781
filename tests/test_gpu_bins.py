"""Bin assignment (Algorithm 3.1) where only sorted output was looked at.

A sorted output does not show a record that was routed to the wrong bin: the
comparison sort puts it right.  So:
* after a sort whose last pass is split, every final bin's slots in the workspace
  are compared with the labels, lone and batched (guarded and unguarded kernels);
* labels longer than the count field of the marks prefix (L > 30 - log2 Z): the
  permutation of the register-resident kernel equals the generic one's.
"""
import ctypes as C

import pytest

import closed_forms as cf
from paper_2008_01765_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2008_01765_amd import bos  # noqa: E402


def _align(x):
    return (x + 255) // 256 * 256


def _check_bins(ws, at, n, rec, z, k, seed):
    """The bins that the split last pass left at workspace offset `at`: bin b's
    first loads[b] slots hold exactly the records of label b (payload = index)."""
    plan = bos.plan(n, rec, z=z, k=k, min_security_bits=0)
    B, L, P = plan["buckets"], plan["levels"], len(plan["passes"])
    assert P >= 2
    lab = bos.debug_labels(n, L, seed).to(torch.int64)
    # the last pass writes slot array (P - 1) mod 2
    at += ((P - 1) & 1) * _align(B * z * rec)
    dt = torch.int32 if rec == 8 else torch.int64
    slots = ws[at:at + B * z * rec].view(dt).view(B, z, 2)
    loads = torch.bincount(lab, minlength=B)
    held = torch.arange(z, device="cuda")[None, :] < loads[:, None]
    idx = slots[..., 1][held].to(torch.int64)
    b = torch.arange(B, device="cuda")[:, None].expand(B, z)[held]
    assert torch.equal(torch.sort(idx).values, torch.arange(n, device="cuda"))
    assert torch.equal(lab[idx], b)


def _first_seed(n, L, z):
    return next(s for s in range(1, 200) if cf.first_overflow(n, cf.labels(s, 0, n, L), 1 << L, L, z)[0] < 0)


CASES = [(32, 2), (256, 1), (256, 2), (256, 3), (512, 1), (512, 2), (512, 3), (512, 4), (1024, 1), (1024, 2)]


@pytest.mark.parametrize("rec", [8, 16])
@pytest.mark.parametrize("z,k", CASES + [(16, 3), (64, 4), (128, 3), (2048, 1)])
def test_bins_of_a_sort(rec, z, k):
    for n in (8 * z * 2 - 3, 40 * z + 7):
        L = bos.plan(n, rec, z=z, k=k, min_security_bits=0)["levels"]
        seed = _first_seed(n, L, z)
        p = bos.params(seed, z, k, min_security_bits=0)
        ws = torch.empty(bos.workspace_bytes(n, rec, p), dtype=torch.uint8, device="cuda")
        x = bos.from_numpy(inputs.records(n, rec, 90))
        out = torch.empty_like(x)
        assert bos.lib().bos_sort(x.data_ptr(), out.data_ptr(), n, rec, C.byref(p), ws.data_ptr(), ws.numel(),
                                  None, None) == bos.OK
        _check_bins(ws, 0, n, rec, z, k, seed)


@pytest.mark.parametrize("rec", [8, 16])
@pytest.mark.parametrize("z,k", CASES)
def test_bins_of_a_batch(rec, z, k):
    # plans of two passes and more, with partial groups
    sizes = [(z << k) + 1, 16 * z * (1 << k) // 2 - 3, 40 * z + 7, 100 * z + 13]
    seeds = [_first_seed(n, bos.plan(n, rec, z=z, k=k, min_security_bits=0)["levels"], z) for n in sizes]
    p = bos.params(0, z, k, min_security_bits=0)
    xs = [bos.from_numpy(inputs.records(n, rec, 91 + i)) for i, n in enumerate(sizes)]
    outs = [torch.empty_like(x) for x in xs]
    arr = (bos.Instance * len(sizes))()
    ns = (C.c_uint64 * len(sizes))(*sizes)
    for i, (x, o) in enumerate(zip(xs, outs)):
        arr[i].in_, arr[i].out, arr[i].n, arr[i].seed = x.data_ptr(), o.data_ptr(), sizes[i], seeds[i]
    nb = bos.lib().bos_batched_workspace_bytes(ns, len(sizes), rec, C.byref(p))
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    status = torch.zeros(len(sizes), dtype=torch.int32, device="cuda")
    assert bos.lib().bos_sort_batched(arr, len(sizes), rec, C.byref(p), ws.data_ptr(), nb, None, status.data_ptr(),
                                      None) == bos.OK
    at = 0
    for n, seed in zip(sizes, seeds):
        _check_bins(ws, at, n, rec, z, k, seed)
        at += _align(bos.workspace_bytes(n, rec, p))


@pytest.mark.parametrize("z", [256, 512, 1024, 2048])
def test_permutation_with_long_labels(z):
    n = (1 << 29) + 1
    x = torch.empty((n, 2), dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x[:, 0] = torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, dtype=torch.int32, device="cuda")
    x[:, 1] = torch.arange(n, dtype=torch.int32, device="cuda")
    assert bos.plan(n, 8, z=z, min_security_bits=0)["levels"] == 31 - z.bit_length() + 1
    a = bos.orp(x, seed=3, z=z, min_security_bits=0)
    b = bos.orp(x, seed=3, z=z, min_security_bits=0, generic=True)
    assert torch.equal(a, b)
    del x, a, b
    bos.release_workspaces()
    torch.cuda.empty_cache()
