"""Regions' totals of the sample attribution: up to 256 regions they come from
the per-PC pass, above from the lifting pass (left out where no metric is
lifted otherwise); integers and alpha identical to the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import log
from test_gpu_samples import assert_samples_parity, run_both

pytestmark = pytest.mark.gpu
DTYPE = np.dtype([("ts", "<u8"), ("ctx", "<u4"), ("region", "<u2"), ("kind", "u1"), ("pad", "u1")])
P = 40


@pytest.mark.parametrize("regions", [7, 300])
@pytest.mark.parametrize("count", [1, 255, 257, 1 << 17, (1 << 17) + 1])
def test_join_blocks(oracle_mod, count, regions):
    """Up to 2^17 samples the join has blocks of 4 waves, beyond of 16."""
    from paper_2609_12299_amd import SAMPLE_DTYPE
    rng = np.random.default_rng(count)
    n = 3000
    r = np.zeros((n, 2), DTYPE)
    r["ctx"] = (np.arange(n) // 500)[:, None]
    r["region"] = rng.integers(0, regions, n)[:, None]
    r["ts"] = (4 * np.arange(n) + 10)[:, None] + np.array([0, 3])
    r["kind"] = [1, 2]
    rec = r.reshape(-1).view(np.uint8).reshape(2 * n, 16)
    s = np.zeros(count, SAMPLE_DTYPE)
    s["ts"] = np.sort(rng.integers(0, 4 * n, count))
    s["ctx_key"], s["pc"] = s["ts"] // 2000, rng.integers(0, P + 1, count)
    weights = rng.integers(0, 9, count).astype(np.uint32)
    log(f"[gpu] {count} samples, {regions} regions")
    g, o = run_both(oracle_mod, rec, regions, s, P, weights=weights)
    assert_samples_parity(g, o, f"{count} samples")


@pytest.mark.parametrize("regions", [1, 64, 255, 256, 257])
def test_region_totals(oracle_mod, regions):
    from paper_2609_12299_amd import SAMPLE_DTYPE
    rng = np.random.default_rng(regions)
    n = 6000
    r = np.zeros((n, 2), DTYPE)
    r["ctx"] = (np.arange(n) // 500)[:, None]
    r["region"] = rng.integers(0, regions, n)[:, None]
    r["ts"] = (4 * np.arange(n) + 10)[:, None] + np.array([0, 3])
    r["kind"] = [1, 2]
    rec = r.reshape(-1).view(np.uint8).reshape(2 * n, 16)
    s = np.zeros(5000, SAMPLE_DTYPE)
    s["ts"] = np.sort(rng.integers(0, 4 * n, len(s)))
    s["ctx_key"], s["pc"] = s["ts"] // 2000, rng.integers(0, P + 1, len(s))
    log(f"[gpu] region totals, {regions} regions")
    for m in (None, rng.random((1, P))):
        g, o = run_both(oracle_mod, rec, regions, s, P, metrics=m)
        assert_samples_parity(g, o, f"R={regions}")
