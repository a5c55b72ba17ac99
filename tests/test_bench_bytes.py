"""The byte model of the benchmark charges a step with what it moves: nothing
where the step returns at once."""
from __future__ import annotations

import os
import sys

import numpy as np
import pytest

from paper_2609_12299_amd import attr

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402

N = 1 << 16
COUNTS = dict(n=N, nv=N, nb=N // 2)


def _plan(early, runs, unsorted):
    slots = np.zeros(16, attr._SLOT)
    # four key digits, from the input when the ingest saw it, else from the context-sorted records
    for i in range(4, 8):
        slots[i] = (1, i, 2 if early and i == 4 else 0, 0, 0, N, N, N // 4096)
    if not early and not runs:
        slots[0] = (1, 0, 2, 0, 0, N, N, N // 4096)
    return dict(n_records=N, n_valid=N, n_begin=N // 2, rec_ts_bits=24, rec_ctx_bits=5, rec_wide=0, unsorted=unsorted,
                early=early, n_ev=0, rec_slots=slots, ev_slots=np.zeros(16, attr._SLOT), ev_merge=1, merge_rounds=1,
                merge_end=N, runs=runs, n_runs=1024)


def _bytes(step, plan):
    return bench.byte_model(step, COUNTS, plan, 8, 2, 8, 3)


@pytest.mark.parametrize("runs", [0, 1])
def test_out_of_order_from_the_start(runs):
    """Seen by the ingest (or forced): one sort from the input, with its own tile sums."""
    p = _plan(1, runs, 1)
    assert [_bytes(s, p) for s in ("ctx_sort", "runs_scatter", "tile_sums")] == [0.0, 0.0, 0.0]
    # histograms (16 per record), four passes (16 + 12, then 12 + 12) and the tile sums (12)
    assert _bytes("full_sort", p) == N * (16 + 28 + 3 * 24 + 12)


@pytest.mark.parametrize("unsorted", [0, 1])
def test_context_sort_first(unsorted):
    p = _plan(0, 0, unsorted)
    assert _bytes("ctx_sort", p) == N * 28 and _bytes("runs_scatter", p) == 0 and _bytes("tile_sums", p) == N * 12
    assert _bytes("full_sort", p) == unsorted * N * (8 + 4 * 24 + 12)
    p = _plan(0, 1, unsorted)
    assert _bytes("ctx_sort", p) == 8 * (N // 256) + 44 * 1024
    assert _bytes("runs_scatter", p) == N * 28 and _bytes("tile_sums", p) == N * 4 + 24 * 1024
