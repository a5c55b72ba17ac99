"""Scoped statistics read only the 256-instance granules that may hold instances
in scope, as marked by the ordinal pass, and the chunks inside one context whose
ordinals reach the iteration window, as found by the carry scan; histogram keys
are kept per granule.  Windows at and around chunk (4096) and granule edges, in
the first, inner and last chunks of a context, beyond every ordinal, for one
region, few, the LDS limit (1024) and beyond; bit-exact against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import log
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
