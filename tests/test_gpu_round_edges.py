"""The single-launch round at the edges of its work split, against the oracle.

Slices of one tile per wave, of exactly one LDS batch of logits (40 tiles) and
of one tile more; every branching factor at which a path changes (one child,
the record's three keys, the candidate pruning from k' = 12); many requests
with a keeper each; ranks that leave padded chunks.  Two more inputs take the
rare paths: the best tokens of every row in one tile (a slice gives up its
whole record, so the merger reads the full lists) and logits that are all
equal (more candidates than the row phase ranks at once).  The vocabulary is
sliced over few workgroups by the test-only launch override, so that small
vocabularies reach the large slices.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2608_02123_amd import pctree as P
from paper_2608_02123_amd.synth import Workload, make_inputs
import compare as C

pytestmark = pytest.mark.gpu

# V, B, N, k, r, R, dtype, slices at most (0: one per compute unit)
SHAPES = [
    (3 * 8 * 16, 3, 24, 8, 32, 1, "bf16", 3),        # one tile per wave
    (3 * 9 * 16 - 7, 3, 24, 8, 32, 1, "bf16", 3),    # one more, ragged
    (3 * 40 * 16, 4, 40, 8, 64, 1, "bf16", 3),       # exactly one batch of logits
    (3 * 41 * 16 - 3, 4, 40, 8, 64, 1, "bf16", 3),   # one tile in a second batch
    (2 * 90 * 16 + 5, 3, 60, 16, 96, 1, "f32", 2),   # three batches, 16 rows
    (4099, 4, 30, 3, 288, 1, "bf16", 0),             # k' = the record's keys
    (4099, 4, 30, 4, 512, 1, "bf16", 0),             # one more: lists
    (4099, 3, 64, 12, 352, 1, "bf16", 0),            # pruned layers, padded chunks
    (4099, 5, 20, 1, 128, 16, "f32", 0),             # 16 requests, chains
    (2050, 4, 20, 2, 16, 8, "f32", 0),
    (2050, 4, 33, 3, 160, 5, "bf16", 0),             # a wave's rows of two requests
    (9001, 3, 50, 8, 256, 2, "bf16", 0),             # 128 candidates
    (70001, 3, 30, 8, 384, 1, "bf16", 61),           # tiles read again every stage
]


def _run(w, inp, slices=0, mode=P.MODE_PARENT):
    dev = P.device_inputs(inp)
    b = P.TreeBuilder(w.V, w.B, w.N, w.k, w.r, w.R, P.BF16 if w.dtype == "bf16" else P.F32,
                      mask=True, trace=True, mode=mode)
    P.debug_set(round_slices=slices)
    try:
        out = b.run(**dev, check=True)
        torch.cuda.synchronize()
    finally:
        P.debug_set()
    return out


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "V{}B{}N{}k{}r{}R{}{}s{}".format(*s))
def test_edges(shape):
    V, B, N, k, r, R, dt, slices = shape
    print(f"[edges] {shape}", flush=True)
    w = Workload("edge", V=V, B=B, N=N, k=k, r=r, R=R, dtype=dt, peak="uniform", seed=5)
    inp = make_inputs(w)
    out = _run(w, inp, slices)
    reps = C.compare_batch(out, inp, k, N, label=f"edges {shape}")
    assert all(rep["exact"] or rep["identical"] for rep in reps), reps


@pytest.mark.parametrize("k", [4, 8, 16])
@pytest.mark.parametrize("mode", ["parent", "shared", "independent"])
def test_best_tokens_in_one_tile(k, mode):
    """The 14 best tokens of every depth share a tile: more than a record holds."""
    print(f"[edges] one tile k={k} {mode}", flush=True)
    w = Workload("tile", V=5000, B=4, N=60, k=k, r=64, R=1, dtype="bf16", peak="none", seed=6)
    inp = make_inputs(w)
    inp["L"][:, :, 1601:1615] += np.float32(32.0) + 4 * np.arange(14, dtype=np.float32)
    inp["L"] = torch.from_numpy(inp["L"]).bfloat16().float().numpy()
    m = {"parent": P.MODE_PARENT, "shared": P.MODE_SHARED, "independent": P.MODE_INDEPENDENT}[mode]
    out = _run(w, inp, mode=m)
    reps = C.compare_batch(out, inp, k, w.N, mode=mode, label=f"one tile k={k} {mode}")
    # (parent-independent scores tie exactly: a + b = b + a across parents)
    assert all(rep["exact"] or rep["identical"] for rep in reps), reps


@pytest.mark.parametrize("V,slices", [(3000, 0), (3000, 2), (2 * 41 * 16, 2)])
def test_equal_logits(V, slices):
    """Every logit equal: ties go to the lowest token, on every path."""
    print(f"[edges] equal logits V={V} slices={slices}", flush=True)
    w = Workload("flat", V=V, B=3, N=40, k=8, r=32, R=1, dtype="f32", peak="none", seed=7,
                 sigma_L=0.0, sigma_W=0.0)
    inp = make_inputs(w)
    out = _run(w, inp, slices)
    reps = C.compare_batch(out, inp, w.k, w.N, label="equal logits")
    assert all(rep["identical"] for rep in reps), reps


def test_abandoned_round_of_many_requests_pads_all():
    """Every keeper gives up when one does: no request keeps a tree."""
    print("[edges] abandoned round, 8 requests", flush=True)
    w = Workload("abort", V=4099, B=4, N=12, k=2, r=32, R=8, dtype="bf16", peak="uniform", seed=8)
    dev = P.device_inputs(make_inputs(w))
    b = P.TreeBuilder(w.V, w.B, w.N, w.k, w.r, w.R, P.BF16, mask=True)
    P.debug_set(wait_ticks=0)
    try:
        out = b.run(**dev)
        torch.cuda.synchronize()
    finally:
        P.debug_set()
    assert (out["count"] == -1).all()
    assert (out["token"] == -1).all() and (out["mask"] == 0).all()
    out = b.run(**dev, check=True)
    assert (out["count"] == w.N).all()  # (a pool of 1 + k + 3 k^2 = 15 nodes)


# V, B, N, k, r, R, dtype: more than 16 frontier rows, base logits at any
# alignment (and vocabularies below one load of four tokens)
WIDE = [(3, 3, 12, 3, 32, 6, "bf16"), (5, 3, 20, 5, 16, 4, "f32"), (1001, 3, 30, 6, 96, 3, "bf16"),
        (1002, 3, 30, 2, 64, 17, "bf16"), (1003, 3, 30, 9, 48, 2, "f32"), (4100, 3, 40, 16, 32, 2, "bf16")]


@pytest.mark.parametrize("shape", WIDE, ids=lambda s: "V{}B{}N{}k{}r{}R{}{}".format(*s))
def test_wide_rows_at_any_alignment(shape):
    V, B, N, k, r, R, dt = shape
    print(f"[edges] wide {shape}", flush=True)
    w = Workload("wide", V=V, B=B, N=N, k=k, r=r, R=R, dtype=dt, peak="uniform", seed=9)
    inp = make_inputs(w)
    out = _run(w, inp)
    reps = C.compare_batch(out, inp, k, N, label=f"wide {shape}")
    assert all(rep["exact"] or rep["identical"] for rep in reps), reps


@pytest.mark.parametrize("k,R,dt", [(8, 2, "f32"), (4, 2, "bf16"), (2, 4, "f32"), (16, 1, "bf16")])
def test_rounds_repeat_bit_for_bit(k, R, dt):
    """No output depends on the order in which workgroups and waves arrive."""
    print(f"[edges] repeats k={k} R={R} {dt}", flush=True)
    w = Workload("rep", V=32000, B=8, N=250, k=k, r=128, R=R, dtype=dt, peak="decay", seed=11)
    dev = P.device_inputs(make_inputs(w))
    b = P.TreeBuilder(w.V, w.B, w.N, w.k, w.r, w.R, P.BF16 if dt == "bf16" else P.F32, mask=True,
                      trace=True)
    g = torch.Generator(device="cuda").manual_seed(12)
    for draw in range(12):
        dev["L"].normal_(0.0, 3.0, generator=g)
        ref = {n: t.clone() for n, t in b.run(**dev, check=True).items()}
        for i in range(8):
            out = b.run(**dev)
            torch.cuda.synchronize()
            for n, t in ref.items():
                assert torch.equal(out[n], t), f"draw {draw} run {i}: {n} differs"


@pytest.mark.parametrize("low", [-np.inf, -np.finfo(np.float32).max, -1e30])
@pytest.mark.parametrize("V,k,R,allowed,slices", [
    (5000, 8, 1, 60, 0),      # most slices are masked whole
    (5000, 3, 2, 40, 0),
    (5000, 16, 1, 30, 0),     # two rows per wave
    (5000, 8, 1, 3, 0),       # fewer unmasked tokens than children
    (3000, 4, 1, 2500, 0),
    (2600, 8, 1, 25, 2),      # two batches of logits per slice
    (12, 8, 1, 5, 0),         # one tile
])
def test_masked_vocabulary(V, k, R, allowed, slices, low):
    """Most base logits at one low value, as constrained decoding masks them: the
    tree of the per-stage launches, and of the oracle where scores are finite."""
    print(f"[edges] masked V={V} k={k} allowed={allowed} {low}", flush=True)
    w = Workload("mask", V=V, B=4, N=40, k=k, r=32, R=R, dtype="f32", peak="none", seed=13)
    inp = make_inputs(w)
    rng = np.random.default_rng(13)
    for q in range(R):
        for d in range(w.B):
            off = rng.permutation(V)[allowed:]
            inp["L"][q, d, off] = np.float32(low)
    out = {n: t.cpu().numpy() for n, t in _run(w, inp, slices).items()}
    P.debug_set(force_multilaunch=True)
    try:
        b = P.TreeBuilder(w.V, w.B, w.N, w.k, w.r, w.R, P.F32, mask=True, trace=True)
        ref = {n: t.cpu().numpy() for n, t in b.run(**P.device_inputs(inp)).items()}
    finally:
        P.debug_set()
    for n, a in ref.items():
        if a.dtype != np.float32:
            np.testing.assert_array_equal(out[n], a, err_msg=n)
        else:  # (a sum of two lowest values overflows in either order of adding)
            np.testing.assert_allclose(out[n], a, rtol=1e-6, atol=C.SCORE_GUARD, err_msg=n)
    assert not np.isnan(out["logprob"]).any()
    if low == -1e30 and allowed >= k:
        reps = C.compare_batch(out, inp, k, w.N, label=f"masked V{V}k{k}")
        assert all(rep["exact"] or rep["identical"] for rep in reps), reps


@pytest.mark.parametrize("k", [1, 8, 16])
def test_two_levels_of_equal_logits(k):
    """More than 64 equal logits above many equal ones: ties to the lowest tokens."""
    print(f"[edges] two levels k={k}", flush=True)
    w = Workload("levels", V=3 * 40 * 16, B=3, N=30, k=k, r=32, R=1, dtype="f32", peak="none",
                 seed=14, sigma_L=0.0, sigma_W=0.0)
    inp = make_inputs(w)
    inp["L"][:, :, 500:1400] = np.float32(2.0)
    inp["L"][:, 1, 700] = np.float32(3.0)
    out = _run(w, inp, 3)
    reps = C.compare_batch(out, inp, k, w.N, label=f"two levels k={k}")
    assert all(rep["identical"] for rep in reps), reps


def test_non_finite_logits_still_end():
    """NaN and infinities among the base logits (outside the contract): the round
    runs to its end at once, as the per-stage launches do."""
    print("[edges] non-finite logits", flush=True)
    w = Workload("nan", V=4000, B=3, N=20, k=8, r=32, R=1, dtype="f32", peak="uniform", seed=15)
    for bad in (np.nan, np.inf, -np.inf):
        for share in (1.0, 0.999, 0.01):
            inp = make_inputs(w)
            inp["L"][np.random.default_rng(1).random(inp["L"].shape) < share] = np.float32(bad)
            out = _run(w, inp)
            assert (out["count"] == w.N).all()
