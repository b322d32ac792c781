"""Timed cases of the library's public calls.

`listed()` names the cases, `draw(rng)` gives another one of the same ranges,
`prepare(case, seed)` builds the inputs and the buffers a program keeps,
`run(state)` makes one pass through the public entry points, `work(case)` is
what a pass cannot do without and `exact(case, seed)` the sorted output by a
library sort.

Sizes follow the repository's own workloads (paper_2008_01765_amd/inputs.py):
2^16 records of 8 bytes, 2^24 of 16 bytes with about sixteen copies of each
key, 2^28 of 8 bytes, batches log-uniform in [2^10, 2^20] and requests
log-uniform in [2^12, 2^24], and odd sizes between them.
"""
import numpy as np
import torch

from paper_2008_01765_amd import autotune, bos, serving

DTYPE = {8: torch.int32, 16: torch.int64}


def listed():
    return [
        # one small sort that a program waits for: launches and host work
        {"name": "sort_r8_1k", "kind": "sort", "rec": 8, "n": 1000, "z": 0, "keys": "uniform", "sync": True},
        # the repository's small workload
        {"name": "sort_r8_64k", "kind": "sort", "rec": 8, "n": 1 << 16, "z": 512, "keys": "uniform", "sync": True},
        # an ordinary table of odd length, 64-bit keys, enqueued without waiting
        {"name": "sort_r16_1m_odd", "kind": "sort", "rec": 16, "n": 1000003, "z": 0, "keys": "uniform",
         "sync": False},
        # the duplicate-heavy workload: about 16 copies of each key
        {"name": "sort_r16_16m_dup", "kind": "sort", "rec": 16, "n": 1 << 24, "z": 0, "keys": "dup", "sync": True},
        # a large odd table whose groups start at unaligned records
        {"name": "sort_r8_50m_odd", "kind": "sort", "rec": 8, "n": 50000017, "z": 0, "keys": "dup", "sync": True},
        # the headline workload
        {"name": "sort_r8_256m", "kind": "sort", "rec": 8, "n": 1 << 28, "z": 512, "keys": "uniform", "sync": True},
        # shuffling a table (random permutation): ordinary odd, 16-byte, large
        {"name": "orp_r8_3m_odd", "kind": "orp", "rec": 8, "n": 3000001, "z": 512, "keys": "uniform", "sync": True},
        {"name": "orp_r16_1m", "kind": "orp", "rec": 16, "n": 1 << 20, "z": 512, "keys": "uniform", "sync": True},
        {"name": "orp_r8_64m", "kind": "orp", "rec": 8, "n": 1 << 26, "z": 512, "keys": "uniform", "sync": True},
        # many uneven sorts in one call
        {"name": "batch_r16_256", "kind": "batch", "rec": 16, "count": 256, "lo": 10, "hi": 18, "z": 0},
        # requests through the continuous-batching server
        {"name": "serve_r16_48", "kind": "serve", "rec": 16, "count": 48, "lo": 12, "hi": 22, "z": 0},
        # records in host memory, streamed through a bounded device workspace
        {"name": "host_sort_r8_16m", "kind": "host_sort", "rec": 8, "n": 1 << 24, "z": 512, "keys": "uniform"},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["sort", "sort", "sort", "orp", "orp", "batch", "serve", "host_sort"])
    rec = rng.choice([8, 16])
    if kind in ("sort", "orp"):
        n = _log_uniform(rng, 1 << 10, 1 << (27 if rec == 8 else 25))
        if rng.random() < 0.6:
            n |= 1
        z = rng.choice([512, 512, 1024]) if kind == "orp" else rng.choice([0, 512, 1024])
        return {"kind": kind, "rec": rec, "n": n, "z": z, "keys": rng.choice(["uniform", "dup"]),
                "sync": rng.random() < 0.7}
    if kind == "batch":
        lo = rng.randrange(10, 13)
        return {"kind": kind, "rec": rec, "count": rng.randrange(8, 257), "lo": lo, "hi": lo + rng.randrange(4, 8),
                "z": 0}
    if kind == "serve":
        return {"kind": kind, "rec": rec, "count": rng.randrange(8, 65), "lo": 12, "hi": rng.randrange(16, 23), "z": 0}
    return {"kind": kind, "rec": rec, "n": _log_uniform(rng, 1 << 20, 1 << (24 if rec == 8 else 23)) | 1,
            "z": 512, "keys": rng.choice(["uniform", "dup"])}


def _sizes(case):
    """Instance sizes of a batch or of a list of requests: log-uniform, fixed
    by the case."""
    if "count" not in case:
        return [case["n"]]
    c, lo, hi = case["count"], case["lo"], case["hi"]
    u = np.random.default_rng([c, lo, hi, case["rec"]]).random(c)
    return [int(v) for v in np.floor(2.0 ** (lo + u * (hi - lo)))]


def _records(n, rec, keys, seed, device):
    """(n, 2) records: keys over their whole width, or about sixteen copies of
    each; payload = index."""
    dt = DTYPE[rec]
    g = torch.Generator(device=device)
    g.manual_seed(seed * 2 + (rec == 16))
    if keys == "dup":
        lo, hi = 0, max(1, n // 16)
    else:
        lo, hi = torch.iinfo(dt).min, torch.iinfo(dt).max
    t = torch.empty((n, 2), dtype=dt, device=device)
    t[:, 0] = torch.randint(lo, hi, (n,), generator=g, dtype=dt, device=device)
    t[:, 1] = torch.arange(n, dtype=dt, device=device)
    return t


def _slices(master, sizes):
    out, at = [], 0
    for s in sizes:
        out.append(master[at:at + s])
        at += s
    return out


def prepare(case, seed):
    kind, rec = case["kind"], case["rec"]
    autotune.install()
    if kind == "host_sort":
        n = case["n"]
        t = bos.pinned_empty((n, 2), DTYPE[rec])
        t.copy_(_records(n, rec, case["keys"], seed, "cpu"))
        p = bos.params(0, case["z"])
        hb = bos.lib().bos_host_workspace_bytes(n, rec, p)
        return {"case": case, "seed": seed, "x": t, "out": bos.pinned_empty((n, 2), DTYPE[rec]),
                "host_ws": bos.pinned_empty((hb,), torch.uint8)}
    sizes = _sizes(case)
    x = _records(sum(sizes), rec, case.get("keys", "uniform"), seed, "cuda")
    st = {"case": case, "seed": seed, "x": x}
    if kind == "serve":
        st["reqs"] = _slices(x, sizes)
        st["server"] = serving.Server(hbm_budget_bytes=16 << 30, z=case["z"])
    else:
        st["out"] = torch.empty_like(x)
        if kind == "batch":
            st["ins"], st["outs"] = _slices(x, sizes), _slices(st["out"], sizes)
            st["seeds"] = [seed + i for i in range(len(sizes))]
    return st


def run(state):
    case, seed = state["case"], state["seed"]
    kind = case["kind"]
    if kind == "sort":
        return bos.sort(state["x"], seed=seed, z=case["z"], out=state["out"], sync=case["sync"])
    if kind == "orp":
        return bos.orp(state["x"], seed=seed, z=case["z"], out=state["out"], sync=case["sync"])
    if kind == "batch":
        bos.sort_batched(state["ins"], state["seeds"], z=case["z"], outs=state["outs"])
        return state["out"]
    if kind == "serve":
        futs = [state["server"].submit(t, seed=seed + i) for i, t in enumerate(state["reqs"])]
        state["server"].run_until_idle()
        return [f.result() for f in futs]
    # the device holds a quarter of a gibibyte of the streamed slots
    return bos.sort_host(state["x"], seed=seed, z=case["z"], out=state["out"], host_ws=state["host_ws"],
                         dev_ws_bytes=1 << 28)


def work(case):
    """Every record read once and written once; the path has no arithmetic on
    floating-point numbers."""
    return {"bytes": 2 * case["rec"] * sum(_sizes(case)), "flops": 0}


def _sorted(t, rec):
    """The records of t (CPU) in unsigned (key, payload) order.  Payloads are
    the indices and ascend, so a stable sort of the unsigned keys is that
    order."""
    a = t.numpy()
    key = a[:, 0].view(np.uint32 if rec == 8 else np.uint64)
    return torch.from_numpy(a[np.argsort(key, kind="stable")])


def exact(case, seed):
    kind, rec = case["kind"], case["rec"]
    sizes = _sizes(case)
    if kind == "orp" or sum(sizes) > 1 << 24:
        return None  # a random permutation, or a library sort of minutes
    dev = "cpu" if kind == "host_sort" else "cuda"
    x = _records(sum(sizes), rec, case.get("keys", "uniform"), seed, dev).cpu()
    outs = [_sorted(t, rec) for t in _slices(x, sizes)]
    if kind == "serve":
        return outs
    return torch.cat(outs) if len(outs) > 1 else outs[0]
