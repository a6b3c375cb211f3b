"""Tree attention at the edges of its work splits, against the float64 oracle.

The direct kernel (few workgroups, at most 24 chunks of 64 slots, eight waves
with chunks of their own), with 16 and 32 rows: admitted ranges that end one
short of, on and one past a chunk, one to three rounds of eight chunks and the
largest cache; requests without slots.  The split runs and their merge (longer
caches).  The one-group and two-group kernels without a split: an odd number of
chunks, requests of very different lengths (taken longest first), and more
requests than that order covers.  Slots past a request's range hold NaN.
"""
from __future__ import annotations

import numpy as np
import pytest

import test_gpu_attention as T

pytestmark = pytest.mark.gpu

D16, D32 = "attn_direct_kernel<{D},1>", "attn_direct_kernel<{D},2>"
ONE, TWO = "attn_kernel<{D},1>", "attn_kernel<{D},2>"

# name, N, Hq, Hkv, D, prefixes, counts, capacity, kernel (test_launches.py checks it)
CASES = [
    ("one short of a chunk", 15, 2, 2, 128, [48], [15], 80, D16),
    ("one chunk", 16, 4, 4, 64, [48], [16], 80, D16),
    ("no split, one chunk", 16, 4, 4, 64, [48], [16], 64, ONE),
    ("one past a chunk", 17, 2, 2, 128, [48], [17], 66, D16),
    ("eight chunks", 11, 6, 2, 64, [501], [11], 600, D16),
    ("eight chunks and a slot", 11, 6, 2, 128, [502], [11], 600, D16),
    ("the largest direct cache, D 128", 45, 28, 4, 128, [1235], [45], 1280, D16),
    ("the largest direct cache, D 64", 45, 28, 4, 64, [1491], [45], 1536, D16),
    ("split runs: one slot more, D 128", 45, 28, 4, 128, [1236], [45], 1281, ONE),
    ("split runs: one slot more, D 64", 45, 28, 4, 64, [1492], [45], 1537, ONE),
    ("split runs: 25 chunks", 45, 28, 4, 128, [1492], [45], 1537, ONE),
    ("split runs: 24 chunks", 45, 28, 4, 128, [1491], [45], 1536, ONE),
    ("32 rows, three rounds", 128, 64, 8, 128, [1400], [128], 1536, D32),
    ("two workgroups per unit", 128, 40, 8, 64, [300, 130], [128, 120], 512, D32),
    ("split runs: too many workgroups", 128, 40, 8, 64, [480, 130], [128, 120], 640, TWO),
    ("32 rows per workgroup", 128, 40, 8, 128, [100, 7], [128, 90], 300, D32),
    # 32 rows and waves with two and three chunks: the V tile is filled again and
    # the running maxima of earlier chunks scale
    ("32 rows, nine chunks", 128, 40, 8, 128, [449], [128], 577, D32),
    ("32 rows, nine chunks, D 64", 128, 40, 8, 64, [448], [128], 576, D32),
    ("32 rows, 17 chunks", 128, 40, 8, 128, [897], [128], 1088, D32),
    ("32 rows, 17 chunks and a slot, D 64", 128, 40, 8, 64, [961], [128], 1090, D32),
    ("32 rows, 24 chunks, D 64", 128, 40, 8, 64, [1408], [128], 1536, D32),
    ("32 rows, 24 chunks less a slot", 121, 40, 8, 128, [1414], [121], 1536, D32),
    ("requests without slots", 20, 8, 2, 64, [0, 30, 0], [0, 0, 20], 70, D16),
    ("split runs", 40, 8, 2, 128, [2100], [40], 2140, ONE),
    ("split runs of two groups", 64, 32, 8, 128, [6000], [64], 6100, TWO),
    ("split runs, D 64, one empty", 33, 6, 3, 64, [3000, 0], [33, 0], 3100, ONE),
    ("no split, mixed lengths", 100, 40, 8, 128, [1, 640, 63, 64, 65, 300, 129, 0],
     [100, 28, 1, 100, 99, 64, 100, 100], 800, TWO),
    ("no split, 70 requests", 9, 4, 2, 64, list(range(0, 210, 3)), [9] * 70, 260, TWO),
    # one group: runs of up to three chunks, and many workgroups
    ("no split, three chunks", 45, 32, 8, 128, [1, 140, 147, 64, 65, 83, 19, 0],
     [45, 45, 45, 19, 44, 45, 45, 45], 192, ONE),
    ("no split, one chunk and a slot, D 64", 45, 32, 8, 64, [20, 19, 0, 3, 5, 7, 11, 20], [45] * 8, 65,
     ONE),
    ("no split, 320 workgroups", 128, 40, 8, 128, [1, 640, 63, 64, 65, 300, 129, 0],
     [128, 28, 1, 100, 99, 64, 128, 100], 768, ONE),
    ("no split, 320 workgroups, 13 chunks", 128, 40, 8, 128, [1, 640, 63, 64, 65, 300, 129, 0],
     [128, 128, 1, 100, 99, 64, 128, 100], 769, TWO),
    ("no split, 320 workgroups, D 64", 128, 40, 8, 64, [200, 640, 63, 64, 65, 300, 129, 0],
     [128] * 8, 768, ONE),
    ("no split, 520 workgroups", 9, 4, 4, 64, list(range(0, 650, 5)), [9] * 130, 833, ONE),
    ("no split, a row per head", 1000, 1, 1, 128, [30] * 16, [1000] * 16, 1030, TWO),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: c[0])
def test_edges(case):
    name, N, Hq, Hkv, D, prefixes, counts, capacity, _ = case
    print(f"[attention edges] {name}", flush=True)
    c = T._case(30, len(prefixes), N, Hq, Hkv, D, prefixes, counts, capacity)
    scale = D ** -0.5
    gpu, att = T._run_gpu(c, scale)
    assert (att.ws_bytes == 0) == name.startswith("no split")
    T._compare(c, gpu, T._oracle(c, scale), name)
    assert np.isfinite(gpu).all()
