"""Scoped statistics are taken by granules of 256 instances and, in large buffers,
read only those that may hold instances in scope, as marked by the ordinal pass, and the chunks inside one context whose
ordinals reach the iteration window, as found by the carry scan; histogram keys
are kept per granule.  Windows at and around chunk (4096) and granule edges, in
the first, inner and last chunks of a context, beyond every ordinal, for one
region, few, the LDS limit (1024) and beyond; bit-exact against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import gpu_run, log
from test_gpu_scope import assert_scope_parity, run_both

pytestmark = pytest.mark.gpu
DTYPE = np.dtype([("ts", "<u8"), ("ctx", "<u4"), ("region", "<u2"), ("kind", "u1"), ("pad", "u1")])
SIZES = [20000, 4096, 300, 4095, 9000, 1]  # instances per context


def _trace(R, seed):
    """Pairs, some nested, some of two regions, and a few BEGINs left open."""
    rng = np.random.default_rng(seed)
    n = sum(SIZES)
    r = np.zeros((n, 2), DTYPE)
    reg = np.where(rng.random(n) < 0.5, rng.integers(0, R, n), rng.integers(0, min(R, 3), n))
    ereg = np.where(rng.random(n) < 0.02, rng.integers(0, R, n), reg)
    for k, kind in ((0, 1), (1, 2)):
        r[:, k]["ts"] = 10 * np.arange(n) + rng.integers(0, 5, n) + 5 * k
        r[:, k]["ctx"] = np.repeat(np.arange(len(SIZES)), SIZES)
        r[:, k]["region"], r[:, k]["kind"] = (reg, ereg)[k], kind
    r = r.reshape(-1)
    swap = np.arange(1, 2 * n - 2, 16)  # E B -> B E: the next pair inside this one
    swap = swap[r["ctx"][swap] == r["ctx"][swap + 1]]
    for f in ("region", "kind"):
        r[f][swap], r[f][swap + 1] = r[f][swap + 1].copy(), r[f][swap].copy()
    keep = (r["kind"] == 1) | (rng.random(2 * n) > 0.0005)
    r = r[keep]
    return r.view(np.uint8).reshape(len(r), 16)


WINDOWS = [(0, 0xFFFFFFFF), (0, 0), (5, 5), (255, 256), (4094, 4097), (6600, 6700), (19990, 0xFFFFFFFF), (30000, 40000)]


@pytest.mark.parametrize("R", [1, 3, 1024, 1025, 4096, 4097])
def test_windows(oracle_mod, R):
    rec = _trace(R, R)
    scopes = [dict(iter_lo=lo, iter_hi=hi) for lo, hi in WINDOWS]
    scopes += [dict(iter_lo=2, iter_hi=700, group_shift=0, group_lo=c, group_hi=c) for c in (0, 3, 4, 9)]
    scopes += [dict(role_mask=3, role_lo=1, role_hi=1), dict(iter_lo=40, iter_hi=50)]
    masks = [None] * (len(scopes) - 1) + [(np.arange(R) % 3 == 0).astype(np.uint8)]
    log(f"[gpu] scope granules R={R}")
    for i, (g, w, nb) in enumerate(run_both(oracle_mod, rec, R, scopes, masks)):
        assert_scope_parity(g, w, nb, f"R={R} scope {scopes[i]}")


@pytest.mark.parametrize("cap", [1 << 22, (1 << 22) + 1])
@pytest.mark.parametrize("R", [3, 1024, 1025, 4096])
def test_windows_of_a_large_buffer(oracle_mod, R, cap):
    """Granules are marked only where the buffer has room for more than 2^22 instances (whatever their number)."""
    import torch

    from paper_2609_12299_amd import scope_statistics
    rec = _trace(R, R)
    g = gpu_run(rec, dict(num_regions=R))
    o = oracle_mod.run(rec, R, 0, None, 0, 0)
    nb = len(g["instances"])
    inst = torch.zeros((cap, 32), dtype=torch.uint8, device="cuda")
    inst[:nb] = torch.from_numpy(g["instances"].view(np.uint8).reshape(nb, 32)).to("cuda")
    excl = torch.zeros(cap, dtype=torch.int64, device="cuda")
    excl[:nb] = torch.from_numpy(g["instance_excl"].view(np.int64)).to("cuda")
    count = torch.tensor([nb], dtype=torch.int64, device="cuda")
    log(f"[gpu] scope granules R={R} in a buffer of {cap}")
    for lo, hi in WINDOWS:
        sc = dict(iter_lo=lo, iter_hi=hi, role_mask=7, role_lo=0, role_hi=3)
        got = scope_statistics(inst, excl, count, R, **sc)
        torch.cuda.synchronize()
        got = {k: v.cpu().numpy() for k, v in got.items() if not k.startswith("_")}
        assert_scope_parity(got, oracle_mod.scope(o["instances"], o["instance_excl"], R, **sc), nb, f"R={R} {sc}")


@pytest.mark.parametrize("R", [1024, 1025])
@pytest.mark.parametrize("n", [256, 257, 1024, 4096, 4097, 32768, 33024, 300000])
def test_few_granules(oracle_mod, n, R):
    """Blocks and granules per wave follow the number of granules: one, a few, one per wave, more."""
    rng = np.random.default_rng(n)
    r = np.zeros((n, 2), DTYPE)
    r["ts"] = np.arange(2 * n).reshape(n, 2) * 3
    r["ctx"] = (np.arange(n) // 700)[:, None]
    r["region"] = rng.integers(0, R, n)[:, None]
    r["kind"] = [1, 2]
    rec = r.reshape(-1).view(np.uint8).reshape(2 * n, 16)
    scopes = [dict(), dict(iter_lo=0, iter_hi=0), dict(group_shift=1, group_lo=1, group_hi=2)]
    log(f"[gpu] scope of {n} instances, R={R}")
    # (a buffer of n instances: half of the records')
    import torch

    from paper_2609_12299_amd import scope_statistics
    g = gpu_run(rec, dict(num_regions=R))
    o = oracle_mod.run(rec, R, 0, None, 0, 0)
    assert len(g["instances"]) == n
    inst = torch.from_numpy(g["instances"].view(np.uint8).reshape(n, 32)).to("cuda")
    excl = torch.from_numpy(g["instance_excl"].view(np.int64)).to("cuda")
    count = torch.tensor([n], dtype=torch.int64, device="cuda")
    for sc in scopes:
        got = scope_statistics(inst, excl, count, R, **sc)
        torch.cuda.synchronize()
        got = {k: v.cpu().numpy() for k, v in got.items() if not k.startswith("_")}
        assert_scope_parity(got, oracle_mod.scope(o["instances"], o["instance_excl"], R, **sc), n, f"R={R} {sc}")
