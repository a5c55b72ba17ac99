"""The probe join up to 256 regions goes by an index over tiles of 4096
instances, above by the sorted reference; the joined probes are sorted in
tiles of 4096 and grouped in tiles of 1024.  Contexts that start at, before and
after tile edges, regions that are rare (many tiles between two of one
context's), groups longer than a tile, iterations past the end and instances of
regions beyond num_regions; all outputs identical to the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import log
from test_gpu_probes import assert_probe_parity, run_both

pytestmark = pytest.mark.gpu
DTYPE = np.dtype([("ts", "<u8"), ("ctx", "<u4"), ("region", "<u2"), ("kind", "u1"), ("pad", "u1")])


def _trace(sizes, R, seed, rare=False):
    """Per context (key 3 c + 1) `size` instances, one after another."""
    rng = np.random.default_rng(seed)
    n = int(sum(sizes))
    r = np.zeros((n, 2), DTYPE)
    ctx = np.repeat(np.arange(len(sizes)) * 3 + 1, sizes)
    reg = rng.integers(0, R, n)
    if rare:
        reg = np.where(rng.random(n) < 0.0003, R - 1, reg % max(R - 1, 1))
    t = np.cumsum(rng.integers(2, 9, n)).astype(np.uint64) * np.uint64(2)
    for k, kind in ((0, 1), (1, 2)):
        r[:, k]["ts"], r[:, k]["ctx"], r[:, k]["region"], r[:, k]["kind"] = t + np.uint64(k), ctx, reg, kind
    return r.reshape(-1).view(np.uint8).reshape(2 * n, 16)


def _probes(m, n_ctx, R, iters, seed, one=False):
    from paper_2609_12299_amd import PROBE_DTYPE
    rng = np.random.default_rng(seed)
    pr = np.zeros(m, PROBE_DTYPE)
    pr["t_start"] = rng.integers(0, 1 << 40, m)
    pr["t_end"] = pr["t_start"] + rng.integers(0, 70000, m).astype(np.uint64)
    pr["ctx_key"] = 4 if one else rng.integers(0, 3 * n_ctx + 2, m)
    pr["iteration"] = 2 if one else np.where(rng.random(m) < 0.01, 0xFFFFFFFF, rng.integers(0, iters, m))
    pr["op_region"] = 0 if one else rng.integers(0, R + 1, m)
    return pr


@pytest.mark.parametrize("R", [1, 2, 255, 256, 257])
@pytest.mark.parametrize("sizes", [[1], [4096, 1, 4095, 4097], [5, 20000, 3], [700] * 30])
def test_tiles(oracle_mod, sizes, R):
    rec = _trace(sizes, R, len(sizes) + R)
    log(f"[gpu] probe index R={R} contexts={len(sizes)}")
    g, o = run_both(oracle_mod, rec, R, _probes(5003, len(sizes), R, max(2, 2 * max(sizes) // R), R))
    assert_probe_parity(g, o, f"R={R}")


def test_rare_region(oracle_mod):
    rec = _trace([60000, 100, 30000], 7, 3, rare=True)
    log("[gpu] probe index: a rare region")
    g, o = run_both(oracle_mod, rec, 7, _probes(20001, 3, 7, 30, 5))
    assert int(o["counters"][2]) > 0
    assert_probe_parity(g, o, "rare")


@pytest.mark.parametrize("m", [1, 1023, 1024, 1025, 4096, 4097, 9000])
def test_one_group(oracle_mod, m):
    rec = _trace([50, 50], 3, 1)
    log(f"[gpu] {m} probes in one group")
    g, o = run_both(oracle_mod, rec, 3, _probes(m, 2, 3, 3, m, one=True))
    assert int(o["counters"][4]) == 1
    assert_probe_parity(g, o, f"m={m}")


def test_fewer_regions_than_the_run(oracle_mod):
    """Instances of regions beyond num_regions are joined by nothing."""
    import torch

    from paper_2609_12299_amd import RegionAttribution, join_probes
    rec = _trace([9000, 4000], 20, 2)
    pr = _probes(3000, 2, 5, 400, 8)
    ra = RegionAttribution(20, max_records=len(rec))
    out = ra.run(torch.from_numpy(rec.reshape(-1)).to("cuda"))
    pt = torch.from_numpy(pr.view(np.uint8).reshape(-1)).to("cuda")
    log("[gpu] probe index: 5 regions of 20")
    g = {k: v.cpu().numpy() for k, v in join_probes(out["instances"], out["counters"][4:5], pt, 5).items()
         if not k.startswith("_")}
    ra.close()
    assert_probe_parity(g, oracle_mod.probes(oracle_mod.run(rec, 20)["instances"], 5, pr), "5 of 20")
