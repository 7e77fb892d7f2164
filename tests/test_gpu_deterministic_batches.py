"""The deterministic operator on meshes with full and partly filled cell
batches at every degree: bitwise repeatable, equal to the 64-bit evaluation of
the timed cases, and not many times slower than the default one (its cells are
added in groups that share no DoF, not one by one).

Tolerances as for the operator elsewhere: 1e-12 (FP64), relative in the
2-norm; FP32 5e-7: inputs, outputs and the batches' partial sums are rounded
to FP32 (8 partial sums at most, 1e-7 each in the worst case), the arithmetic
inside a batch is FP64.
"""
import pytest
import torch

from paper_2203_12292_amd import mfmg
from perf import cases

pytestmark = pytest.mark.gpu
TOL = {"f64": 1e-12, "f32": 5e-7}
MESHES = [("spheres", 3, 1, 1), ("ball", 4, 1, 2)]


def level_and_input(mesh, k, dtype, nv):
    case = cases._case("vmult", *mesh, k, dtype, nv, "h_then_p")
    m = mfmg.Mesh(cases._desc(case))
    S = mfmg.Solver(m, k, mfmg.SCHEME_H_THEN_P, level_dtypes=[cases.CODES[dtype]], max_rhs=nv, deterministic=True)
    return case, S, S.n_levels - 1, cases.prepare(case, 5)


@pytest.mark.parametrize("mesh", MESHES)
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("dtype,nv", [("f64", 1), ("f32", 1), ("f64", 3), ("f32", 8)])
def test_repeatable_and_right(mesh, k, dtype, nv):
    case, S, top, st = level_and_input(mesh, k, dtype, nv)
    y = [S.vmult(top, torch.empty_like(st["y"]), st["x"], nv) for _ in range(5)]
    assert all(torch.equal(y[0], z) for z in y[1:])
    want = cases.exact(case, 5)
    assert float((y[0].double() - want).norm() / want.norm()) <= TOL[dtype]


@pytest.mark.parametrize("k", [1, 2])
def test_costs_a_few_default_applications(k):
    case, S, top, st = level_and_input(("spheres", 3, 0, 2), k, "f64", 1)

    def microseconds(solver):
        best = float("inf")
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(50):
                solver.vmult(top, st["y"], st["x"])
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3 / 50)
        return best

    slow, fast = microseconds(S), microseconds(st["solver"])
    print(f"Q{k}: deterministic {slow:.1f} us, default {fast:.1f} us", flush=True)
    assert slow <= 6 * fast
