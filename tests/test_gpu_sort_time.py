"""The passes of a sort share one kernel, in which a pass starts when the one
before it has ended everywhere.  That wait must not hold up the blocks still at
work: a pass in the middle of a sort costs no more than one that runs alone."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import log

pytestmark = pytest.mark.gpu
DTYPE = np.dtype([("ts", "<u8"), ("ctx", "<u4"), ("region", "<u2"), ("kind", "u1"), ("pad", "u1")])


def _step_ms(ts, ctx, step, **kw):
    """Shortest of ten times of one step (ms), and the passes that the run's sorts made."""
    import torch

    from paper_2609_12299_amd import RegionAttribution
    n = len(ts)
    r = np.zeros(n, DTYPE)
    r["ts"], r["ctx"] = ts, ctx
    r["kind"] = 1 + np.arange(n) % 2
    rec = torch.from_numpy(r.view(np.uint8)).to("cuda")
    ra = RegionAttribution(4, max_records=n, **kw)
    for _ in range(2):
        ra.run(rec)
    ra.set_timing(True)
    for _ in range(10):
        ra.run(rec)
    ms = min(t for name, t in ra.kernel_times() if name == step)
    active = [bool(s["active"]) for s in ra.plan()["rec_slots"]]
    ra.close()
    return ms, sum(active[:4]), sum(active[4:])


@pytest.mark.parametrize("n", [1 << 21, 1 << 22])
def test_inner_pass(n):
    rng = np.random.default_rng(3)
    # one pass by context over the raw records, with nothing to wait for
    alone, ctx_passes, _ = _step_ms(np.arange(n, dtype=np.uint64), rng.integers(0, 200, n), "ctx_sort",
                                    force_record_radix=True)
    assert ctx_passes == 1
    three, _, p3 = _step_ms(rng.integers(0, 1 << 24, n, dtype=np.uint64), 0, "full_sort")
    six, _, p6 = _step_ms(rng.integers(0, 1 << 48, n, dtype=np.uint64), 0, "full_sort")
    assert (p3, p6) == (3, 6)
    inner = (six - three) / 3
    log(f"[gpu] {n} records: a pass alone {alone * 1e3:.1f} us, inside a sort {inner * 1e3:.1f} us")
    assert inner < 1.3 * alone
