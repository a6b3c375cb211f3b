"""Tree attention at the edges of its work splits, against the float64 oracle.

The direct kernel (few workgroups, at most 24 chunks of 64 slots, eight waves
with chunks of their own): admitted ranges that end one short of, on and one
past a chunk, a round of eight chunks and the largest cache; 15, 16, 17 and 33
rows; requests without slots.  The split runs and their merge (longer caches).
The two-group kernel without a split: an odd number of chunks, requests of very
different lengths (taken longest first), and more requests than that order
covers.  Slots past a request's range hold NaN.
"""
from __future__ import annotations

import numpy as np
import pytest

import test_gpu_attention as T

pytestmark = pytest.mark.gpu

# name, N, Hq, Hkv, D, prefixes, counts, capacity
CASES = [
    ("one short of a chunk", 15, 2, 2, 128, [48], [15], 80),
    ("one chunk", 16, 4, 4, 64, [48], [16], None),
    ("one past a chunk", 17, 2, 2, 128, [48], [17], None),
    ("eight chunks", 11, 6, 2, 64, [501], [11], 600),
    ("eight chunks and a slot", 11, 6, 2, 128, [502], [11], 600),
    ("the largest direct cache", 45, 28, 4, 128, [1491], [45], 1536),
    ("one slot more: split runs", 45, 28, 4, 128, [1492], [45], 1537),
    ("two workgroups per unit", 128, 40, 8, 64, [300, 130], [128, 120], 512),
    ("too many workgroups: split runs", 128, 40, 8, 64, [480, 130], [128, 120], 640),
    ("32 rows per workgroup", 128, 40, 8, 128, [100, 7], [128, 90], 300),
    ("requests without slots", 20, 8, 2, 64, [0, 30, 0], [0, 0, 20], 60),
    ("split runs", 40, 8, 2, 128, [2100], [40], None),
    ("split runs, D 64, one empty", 33, 6, 3, 64, [3000, 0], [33, 0], 3100),
    ("no split, mixed lengths", 100, 40, 8, 128, [1, 640, 63, 64, 65, 300, 129, 0],
     [100, 28, 1, 100, 99, 64, 100, 100], 800),
    ("no split, 70 requests", 9, 4, 2, 64, list(range(0, 210, 3)), [9] * 70, 260),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: c[0])
def test_edges(case):
    name, N, Hq, Hkv, D, prefixes, counts, capacity = case
    print(f"[attention edges] {name}", flush=True)
    c = T._case(30, len(prefixes), N, Hq, Hkv, D, prefixes, counts, capacity)
    scale = D ** -0.5
    gpu, att = T._run_gpu(c, scale)
    assert (att.ws_bytes == 0) == name.startswith("no split") or capacity is None or capacity <= 64
    T._compare(c, gpu, T._oracle(c, scale), name)
    assert np.isfinite(gpu).all()
