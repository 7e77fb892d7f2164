"""A smoothing step on FP64 vectors moves twice the bytes of one on FP32
vectors, with the same arithmetic inside the cells: it takes no more than
twice the time (degree 3, 270,000 cells, 7.3 million DoFs)."""
import pytest
import torch

from perf import cases

pytestmark = pytest.mark.gpu


def test_fp64_step_within_twice_the_fp32_step():
    t = {}
    for dtype in ("f64", "f32"):
        st = cases.prepare(cases._case("smooth", "octant", 1, 0, 7, 3, dtype, 1, "h"), 3)
        cases.run(st)
        best = float("inf")
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                cases.run(st)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3 / 20)
        t[dtype] = best
    print(f"Q3 smoothing step: FP64 {t['f64']:.0f} us, FP32 {t['f32']:.0f} us", flush=True)
    assert t["f64"] <= 2 * t["f32"]
