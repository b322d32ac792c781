"""Helpers shared by the GPU tests (no method arithmetic here)."""
import contextlib

import numpy as np


def bucket_sets_equal(rec_a, tag_a, rec_b, tag_b):
    """True when every bucket of two slot arrays (B, Z, 2) / (B, Z) holds the same
    multiset of real (record, tag) slots and the same number of dummies, and all
    dummies are canonical (zero record)."""
    def canon(rec, tag):
        B, Z = tag.shape
        real = tag != 0xFFFFFFFF
        bidx = np.broadcast_to(np.arange(B)[:, None], (B, Z))[real]
        t = tag[real].astype(np.uint64)
        k = rec[..., 0][real].astype(np.uint64)
        p = rec[..., 1][real].astype(np.uint64)
        o = np.lexsort((p, k, t, bidx))
        dummies_ok = bool(np.all(rec[~real] == 0))
        return bidx[o], t[o], k[o], p[o], real.sum(axis=1), dummies_ok
    a, b = canon(rec_a, tag_a), canon(rec_b, tag_b)
    return all(np.array_equal(x, y) for x, y in zip(a[:5], b[:5])) and a[5] and b[5]


def record_checksum(a):
    """Order-independent 64-bit checksum of a record array (sum and xor of a mix)."""
    with np.errstate(over="ignore"):
        k = a[:, 0].astype(np.uint64)
        p = a[:, 1].astype(np.uint64)
        z = k * np.uint64(0x9E3779B97F4A7C15) ^ (p + np.uint64(0x632BE59BD9B4E019))
        z ^= z >> np.uint64(29)
        z *= np.uint64(0xBF58476D1CE4E5B9)
        z ^= z >> np.uint64(32)
        return int(z.sum(dtype=np.uint64)), int(np.bitwise_xor.reduce(z)) if z.size else 0


def _unsigned_order_i64(col):
    """int32 / int64 record column (bits taken as unsigned) as int64 values
    with the unsigned order (torch has no 64-bit unsigned sort)."""
    import torch
    if col.dtype == torch.int32:
        return col.to(torch.int64) & 0xFFFFFFFF
    return col ^ torch.iinfo(torch.int64).min


def torch_sorted_records(t):
    """Records of a CUDA tensor sorted by (key, payload), unsigned, with torch's
    library sort."""
    import torch
    k = _unsigned_order_i64(t[:, 0])
    p = _unsigned_order_i64(t[:, 1])
    idx = torch.argsort(p, stable=True)
    idx = idx[torch.argsort(k[idx], stable=True)]
    return t[idx]


def torch_is_sorted(t):
    """True when the records of a CUDA tensor are in (key, payload) order."""
    k = _unsigned_order_i64(t[:, 0])
    p = _unsigned_order_i64(t[:, 1])
    if t.shape[0] < 2:
        return True
    ok = (k[1:] > k[:-1]) | ((k[1:] == k[:-1]) & (p[1:] >= p[:-1]))
    return bool(ok.all())


@contextlib.contextmanager
def trace_digests(slots):
    """With the digest build (see test_gpu_trace.py) loaded: a function that
    calls fn with zeroed digest buffers of `slots` slots and returns (status,
    routing digests, comparison-sort digests)."""
    import torch
    from paper_2008_01765_amd import bos
    with bos.using_library(bos.TRACE_LIB_PATH) as L:
        bufs = [torch.zeros(slots, dtype=torch.int64, device="cuda") for _ in range(2)]
        assert L.bos_trace_bind(bufs[0].data_ptr(), bufs[1].data_ptr(), slots) == bos.OK

        def run(fn, *args, **kw):
            for b in bufs:
                b.zero_()
            torch.cuda.synchronize()
            st = bos.OK
            try:
                fn(*args, **kw)
            except bos.BosError as e:
                st = e.status
            torch.cuda.synchronize()
            return st, bufs[0].clone(), bufs[1].clone()

        try:
            yield run
        finally:
            L.bos_trace_bind(None, None, 0)
