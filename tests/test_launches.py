"""What calls launch, checked without a GPU (launches.py)."""
from __future__ import annotations

import pytest

from paper_2608_02123_amd import pctree as P
import launches as X

# V, B, N, k, r, R, dtype, mode
NARROW = [151936, 16, 64, 8, 256, 1, P.BF16, 0]
WIDE = [151936, 4, 64, 16, 512, 8, P.BF16, 0]


def _names(result):
    assert result["status"] == P.OK
    return [k[0] for k in result["kernels"]]


def test_round_forms(tmp_path):
    r = X.record([{"round": NARROW}, {"round": WIDE}], P.LIB_PATH, tmp_path)
    assert _names(r[0]) == ["clear_kernel", "round_kernel<1,8,1>"]
    # every workgroup has a compute unit of its own
    assert r[0]["kernels"][1][1] <= 256
    assert _names(r[1]) == (["probe_kernel", "prologue_kernel"]
                            + ["head_thr_kernel<1,16,16>", "mergesel_kernel<16>"] * 4
                            + ["emit_kernel"])


@pytest.mark.parametrize("fail", [(1, 0), (3, 0), (0, 1), (0, 2)])
def test_a_failed_query_is_asked_again(fail, tmp_path):
    """A device query that fails costs that call the single launch, not the
    process; the call itself still succeeds."""
    n = sum(fail)
    r = X.record([{"reset": [256, *fail]}, {"round": WIDE}] + [{"round": NARROW}] * (n + 2),
                 P.LIB_PATH, tmp_path)[1:]
    assert "head_thr_kernel<1,16,16>" in _names(r[0])
    assert "prologue_kernel" in _names(r[1])  # (per-stage launches)
    for call in r[1:]:
        _names(call)
    assert _names(r[-2])[-1] == _names(r[-1])[-1] == "round_kernel<1,8,1>"
