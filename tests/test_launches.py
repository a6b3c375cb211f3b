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


def _attention(tmp_path, shapes, cus=256):
    calls = [{"reset": [cus, 0, 0]}] + [{"attention": list(s)} for s in shapes]
    return X.record(calls, P.LIB_PATH, tmp_path)[1:]


def test_attention_kernels_over_the_range(tmp_path):
    """Every layer takes the kernel that the rule names, with a workgroup for every
    block of rows and no launch that the device refuses."""
    shapes = [(R, N, Hq, Hkv, D, C) for D in (64, 128)
              for Hq, Hkv in ((32, 8), (40, 8), (16, 16), (28, 4), (2, 2), (71, 1))
              for R in (1, 2, 8, 70) for N in (1, 16, 45, 128, 1024)
              for C in (1, 64, 65, 512, 513, 1088, 1280, 1281, 1536, 1537, 4096)
              if R * N * Hq * D <= 1 << 31]
    seen = set()
    for (R, N, Hq, Hkv, D, C), r in zip(shapes, _attention(tmp_path, shapes)):
        names = _names(r)
        g, heads, chunks = Hq // Hkv, R * Hkv, -(-C // 64)
        rows, base = N * g, R * Hkv * -(-N * g // 128)
        runs = min(-(-128 // base), chunks, 32) if base < 128 else 1
        per = -(-chunks // runs)
        runs = -(-chunks // per)
        direct = runs > 1 and chunks <= 24 and not (D == 128 and chunks > 20 and per <= 4)
        if direct and heads * -(-rows // 16) <= 256:
            want, block = [f"attn_direct_kernel<{D},1>"], 16
        elif direct and (heads * -(-rows // 32) <= 256 or chunks <= 8):
            want, block = [f"attn_direct_kernel<{D},2>"], 32
        else:
            groups = 1 if per <= 3 or base > (256 if chunks <= 12 else 512) else 2
            want, block = [f"attn_kernel<{D},{groups}>"], 128
            heads *= runs
            if runs > 1:
                want.append(f"attn_merge_kernel<{D}>")
        assert names == want, (R, N, Hq, Hkv, D, C)
        # whole rounds of the eight XCDs, every block of rows among them
        assert r["kernels"][0][1] == -(-heads // 8) * 8 * -(-rows // block)
        assert r["kernels"][0][3] <= 24 * 1024  # (the mask rows, past the tiles)
        seen.add((want[0], len(want)))
    assert len(seen) == 2 * 6  # every kernel, split and not, for both head sizes


def test_attention_edge_cases_take_the_kernels_they_name(tmp_path):
    import test_gpu_attention_edges as E

    shapes = [(len(c[5]), c[1], c[2], c[3], c[4], c[7]) for c in E.CASES]
    for case, r in zip(E.CASES, _attention(tmp_path, shapes)):
        assert _names(r)[0] == f"{case[8].format(D=case[4])}", case[0]
        assert (len(r["kernels"]) == 2) == case[0].startswith("split runs"), case[0]
