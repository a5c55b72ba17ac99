"""The sorts of the records take different routes: contexts in time order
(context sort only), shuffled buffers (noticed while the records are read: one
sort from the input), buffers out of order only where that reading does not
look (noticed after the context sort), with keys that fit 64 bits and keys that
do not, over runs and over records.  Each must match the oracle bit for bit,
at the edges of the 4096-element sort tiles and where a sort clears its own
look-back words (beyond 2^25 records)."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import assert_parity, gpu_run, log, oracle_run

pytestmark = pytest.mark.gpu
DTYPE = np.dtype([("ts", "<u8"), ("ctx", "<u4"), ("region", "<u2"), ("kind", "u1"), ("pad", "u1")])
P = dict(num_regions=6, num_classes=2, region_class=np.array([0, 1, 0, 1, 0xFF, 0], np.uint8), group_shift=2,
         num_groups=40)


def _records(n, order, wide, seed):
    rng = np.random.default_rng(seed)
    n_ctx = 37
    r = np.zeros(n, DTYPE)
    r["ctx"] = rng.integers(0, n_ctx, n) if order != "late" else (np.arange(n) // 256) % n_ctx
    r["ts"] = np.cumsum(rng.integers(0, 40, n))
    r["region"] = rng.integers(0, 7, n)  # one region out of range
    r["kind"] = rng.integers(1, 3, n)
    if order == "shuffled":
        r = r[rng.permutation(n)]
    elif order == "late":
        # one context per 256-record chunk: times go back only in the last rows of a chunk
        for c in range(0, n - 255, 512):
            r["ts"][c + 200:c + 256] = r["ts"][c + 200:c + 256][::-1]
    if wide:
        r["ctx"] = r["ctx"] * np.uint32(0x6000000) + np.uint32(3)
        r["ts"] = r["ts"] + (r["ctx"] % np.uint32(5)).astype(np.uint64) * np.uint64(1 << 60)
    return r.view(np.uint8).reshape(n, 16)


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("order", ["in_order", "shuffled", "late"])
@pytest.mark.parametrize("n", [1, 300, 4095, 4096, 4097, 70001])
def test_routes(oracle_mod, n, order, wide):
    rec = _records(n, order, wide, n + 3)
    log(f"[gpu] sort route n={n} order={order} wide={wide}")
    g = gpu_run(rec, P, with_plan=True)
    plan = g.pop("_plan")
    if n >= 4095:
        assert plan["unsorted"] == (0 if order == "in_order" else 1)
        assert plan["rec_wide"] == int(wide)
    assert_parity(g, oracle_run(oracle_mod, rec, P), what=f"{order} wide={wide}")
    assert_parity(gpu_run(rec, P, force_full=True, force_event=True), oracle_run(oracle_mod, rec, P),
                  what=f"{order} wide={wide}, both sorts forced")


@pytest.mark.parametrize("K", [1, 3, 8])
@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 1, (1 << 20) + 4096])
def test_event_sort_split(oracle_mod, n, K):
    """Up to 2^20 records the events are sorted and swept by one kernel, beyond by two."""
    rec = _records(n, "late", False, K)
    p = dict(P, num_classes=K, region_class=np.array([0, 1 % K, 2 % K, 7 % K, 0xFF, K - 1], np.uint8))
    log(f"[gpu] event sort of {n} records, {K} classes")
    g = gpu_run(rec, p, force_event=True, with_plan=True)
    plan = g.pop("_plan")
    assert plan["ev_merge"] == 0 and plan["n_ev"] > 0
    assert_parity(g, oracle_run(oracle_mod, rec, p), what=f"n={n} K={K}")


@pytest.mark.timeout(400)
@pytest.mark.parametrize("order,radix", [("in_order", True), ("shuffled", False), ("late", False)])
def test_beyond_init_clear(oracle_mod, order, radix):
    n = (1 << 25) + 4097
    rec = _records(n, order, False, 9)
    log(f"[gpu] sort route n={n} order={order} radix={radix}")
    g = gpu_run(rec, P, force_radix=radix, with_plan=True)
    assert g.pop("_plan")["unsorted"] == (0 if order == "in_order" else 1)
    assert_parity(g, oracle_run(oracle_mod, rec, P), what=order)
