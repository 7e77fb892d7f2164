"""The operator at degrees 5 and 6 on levels with few cell batches (a line of
nodes per lane) and with more of them (a plane per lane, with level-wide blocks
larger than most batches need), plain and fused, against the 64-bit evaluation
of the timed cases; and a small level of degree 6 takes little longer than one
of degree 4.

Tolerances, relative in the 2-norm: FP64 1e-12 as elsewhere.  FP32 5e-7:
input, output and the partial sums of at most 8 batches are rounded to FP32
(6e-8 each), the arithmetic inside a batch is FP64; a smoothing step rounds x
and d in each of its three applications, twice that.  bfloat16: the output's
rounding 2^-9, a step's six roundings and their way through the operator 2e-2.
"""
import pytest
import torch

from perf import cases

pytestmark = pytest.mark.gpu
TOL = {"vmult": {"f64": 1e-12, "f32": 5e-7, "bf16": 4e-3}, "smooth": {"f64": 1e-12, "f32": 1e-6, "bf16": 2e-2}}
MESHES = [("ball", 2, 0, 2), ("ball", 4, 0, 3), ("octant", 1, 0, 4)]


@pytest.mark.parametrize("mesh", MESHES)
@pytest.mark.parametrize("k", [5, 6])
@pytest.mark.parametrize("op,dtype,nv", [("vmult", "f64", 1), ("vmult", "f32", 1), ("vmult", "f64", 3),
                                         ("vmult", "f32", 8), ("vmult", "bf16", 2), ("smooth", "f64", 1),
                                         ("smooth", "f32", 1), ("smooth", "bf16", 1), ("smooth", "f64", 2)])
def test_right(mesh, k, op, dtype, nv):
    case = cases._case(op, *mesh, k, dtype, nv, "h" if mesh[1] == 1 else "h_then_p")
    got, want = cases.run(cases.prepare(case, 3)), cases.exact(case, 3)
    assert float((got.double() - want).norm() / want.norm()) <= TOL[op][dtype]


def microseconds(call):
    call()
    best = float("inf")
    for _ in range(6):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(50):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / 50)
    return best


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_small_level_of_degree_6_against_degree_4(dtype):
    t = {}
    for k in (4, 6):
        st = cases.prepare(cases._case("smooth", "spheres", 3, 0, 2, k, dtype, 1, "h_then_p"), 3)
        t[k] = microseconds(lambda: cases.run(st))
    print(f"smoothing step on 832 cells, {dtype}: Q4 {t[4]:.1f} us, Q6 {t[6]:.1f} us", flush=True)
    assert t[6] <= 1.3 * t[4]
