"""bench.py's account of the launches that ran: per-launch figures of a call
that mixes launches of four, two and one steps, and a warm-up that leaves no
kernel's first launch to the timed region."""
import os
import sys

import pytest

ROOT = os.path.join(os.path.dirname(__file__), "..")
sys.path.insert(0, ROOT)
import bench  # noqa: E402

N = 16384


def line(split, ms=1.6, form="f32", variant="B"):
    return bench.roofline(form, variant, N, {**split, "tile4": None}, 16, ms)


def test_figures_are_those_of_the_launches(monkeypatch):
    traffic = {"f32_kbcB_16384_fused4": 196.0, "f32_kbcB_16384_fused2": 202.0, "f32_kbcB_16384": 193.0}
    valu = {"f32_kbcB_16384_fused4": 206.0, "f32_kbcB_16384_fused2": 186.0}
    monkeypatch.setattr(bench, "measured_traffic",
                        lambda key, section="step", field="bytes_per_launch":
                        (traffic if field == "bytes_per_launch" else valu).get(key))
    r = line({4: 16, 2: 4, 1: 0})          # 20 steps: four launches of four, two of two
    assert r["launches"] == {"k_step4<f32,KBC-B>": 4, "k_step2<f32,KBC-B,64x16>": 2}
    assert r["steps_per_launch"] == pytest.approx(20 / 6, abs=1e-4) and r["kernel"] == "k_step4<f32,KBC-B>"
    seconds = 1.6e-3 * 20
    assert r["hbm_GBs_per_launch"] == pytest.approx(72 * N * N * 6 / seconds / 1e9, rel=1e-4)
    assert r["achieved"] == pytest.approx(bench.FLOPS_PER_NODE_STEP["f32"] * N * N * 20 / seconds / 1e12, rel=1e-3)
    assert r["traffic"] == round((4 * 196.0 + 2 * 202.0) / 6)
    assert r["valu_instructions_per_node_step"] == pytest.approx((16 * 206.0 + 4 * 186.0) / 20, abs=0.05)
    # a kernel that was not counted: no figure
    assert line({4: 16, 2: 4, 1: 0}, form="f16")["traffic"] is None
    assert "valu_issue_frac" not in line({4: 16, 2: 0, 1: 1})
    # four steps: no launch of four
    r = line({4: 0, 2: 4, 1: 0})
    assert r["steps_per_launch"] == 2 and r["kernel"].startswith("k_step2") and r["traffic"] == 202
    r = line({4: 0, 2: 0, 1: 4})
    assert r["steps_per_launch"] == 1 and r["bound"] == "hbm" and r["traffic"] == 193
    assert line({4: 200, 2: 0, 1: 0})["steps_per_launch"] == 4


def test_kernels_are_loaded_before_the_warm_up(monkeypatch):
    """A call that makes a launch of every kind, before the warm-up."""
    import torch
    calls = []

    class Small:
        def step(self, n):
            calls.append(n)

    monkeypatch.setattr(bench, "make_sim", lambda *a: Small())
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    bench.load_kernels("f32", "B", 1e-4, 3, 32, "cpu")
    assert len(calls) == 1 and calls[0] % 8 == 3      # groups of eight, a pair and a single step
    src = open(os.path.join(ROOT, "bench.py")).read()
    main = src[src.index("def main()"):]
    assert 0 < main.index("load_kernels(") < main.index("time_steps(")
