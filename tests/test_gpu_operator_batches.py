"""The operator, its fused steps and several vectors on meshes with full and
partly filled cell batches at every degree (up to 1,024 cells in a batch at
degree 1, 8 at degree 6; a lane per cell up to degree 2, a lane per plane of
nodes from degree 3), with one, two and three hanging faces and hanging edges,
against the 64-bit torch evaluation of the timed cases.

Tolerances as for the operator elsewhere: 1e-12 (FP64), 2e-5 (FP32), 2e-2
(bfloat16), relative in the 2-norm; the residual of a smoothed vector loses the
digits that b - A x cancels, a factor of 10 here.
"""
import pytest
import torch

from perf import cases

pytestmark = pytest.mark.gpu
TOL = {"f64": 1e-12, "f32": 2e-5, "bf16": 2e-2}


def check(op, mesh, k, dtype, nv, scheme):
    name, n0, g, steps = mesh
    case = cases._case(op, name, n0, g, steps, k, dtype, nv, scheme)
    got = cases.run(cases.prepare(case, 5))
    want = cases.exact(case, 5)
    if op != "descend":
        got, want = (got,), (want,)
    for i, (a, b) in enumerate(zip(got, want)):
        err = float((a.double() - b).norm() / b.norm())
        assert err <= TOL[dtype] * (10 if i else 1), (i, err)


@pytest.mark.parametrize("mesh", [("spheres", 3, 1, 2), ("ball", 4, 1, 2)])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("dtype,nv", [("f64", 1), ("f32", 8), ("f64", 3), ("bf16", 2)])
def test_vmult(mesh, k, dtype, nv):
    check("vmult", mesh, k, dtype, nv, "h_then_p")


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_fused_steps(k, dtype):
    check("descend", ("shell", 1, 2, 3), k, dtype, 1, "h")
