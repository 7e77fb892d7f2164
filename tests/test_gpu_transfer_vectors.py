"""Transfers of several vectors, on levels small enough that each vector has
wavefronts of its own and large enough that one wavefront takes all vectors:
every vector comes out as it does alone, in FP64, FP32 and the deterministic
mode, for each pair of degrees, and a call on several vectors costs no more
than one call per vector.

Tolerance: the vectors of a call and a vector alone run the same sums in
another order; a value passes six contractions of at most 13 terms (two per
axis, hanging interpolation and sweep) and up to 8 atomic additions, about 90
roundings of the type's unit, relative to the largest entry: 1e-14 x 2 (FP64)
and 1.2e-5 (FP32).
"""
import functools

import pytest
import torch

import synth
from helpers import SCHEME_CODES

pytestmark = pytest.mark.gpu
DTYPES = {"f64": (0, torch.float64, 2e-14), "f32": (1, torch.float32, 1.2e-5)}


@functools.lru_cache(maxsize=2)
def solver(scheme, k, depth, dtype, deterministic):
    from paper_2203_12292_amd import mfmg
    return mfmg.Solver(mfmg.Mesh(synth.octant_mesh(depth)), k, SCHEME_CODES[scheme], level_dtypes=[DTYPES[dtype][0]],
                       max_rhs=8, deterministic=deterministic)


def rand(n, dt, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (2 * torch.rand(n, dtype=torch.float64, device="cuda", generator=g) - 1).to(dt)


@pytest.mark.parametrize("nv", [2, 3, 5, 8])
@pytest.mark.parametrize("dtype,deterministic", [("f64", False), ("f32", False), ("f32", True)])
@pytest.mark.parametrize("scheme,k,depth", [("h", 1, 3), ("h", 2, 6), ("h", 3, 4), ("h", 4, 6), ("h", 5, 4), ("h", 6, 4),
                                            ("h", 6, 6), ("p_then_h", 4, 4), ("p_then_h", 5, 5), ("p_then_h", 6, 3),
                                            ("p_then_h", 6, 5), ("hp", 4, 5), ("hp", 6, 4)])
def test_each_vector_as_alone(scheme, k, depth, dtype, deterministic, nv):
    S = solver(scheme, k, depth, dtype, deterministic)
    _, dt, tol = DTYPES[dtype]
    top = S.n_levels - 1
    n, nc = (S.level_info(l)["n_dofs"] for l in (top, top - 1))
    f, c = rand(n * nv, dt, 1), rand(nc * nv, dt, 2)
    F, C = S.prolongate_add(top, f.clone(), c, nv), S.restrict_add(top, c.clone(), f, nv)
    for v in range(nv):
        f1, c1 = f.view(-1, nv)[:, v].contiguous(), c.view(-1, nv)[:, v].contiguous()
        F1, C1 = S.prolongate_add(top, f1.clone(), c1), S.restrict_add(top, c1.clone(), f1)
        assert float((F.view(-1, nv)[:, v] - F1).abs().max()) <= tol * float(F1.abs().max())
        assert float((C.view(-1, nv)[:, v] - C1).abs().max()) <= tol * float(C1.abs().max())


def microseconds(call, n=100):
    call()
    best = float("inf")
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(n):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / n)
    return best


@pytest.mark.parametrize("k,nv", [(4, 3), (6, 3), (6, 5)])
def test_several_vectors_cost_no_more_than_a_call_each(k, nv):
    S = solver("h", k, 4, "f64", False)
    top = S.n_levels - 1
    n, nc = (S.level_info(l)["n_dofs"] for l in (top, top - 1))
    f, c = (torch.zeros(m * nv, dtype=torch.float64, device="cuda") for m in (n, nc))
    f1, c1 = f[:n], c[:nc]
    for op, args, alone in ((S.restrict_add, (c, f), (c1, f1)), (S.prolongate_add, (f, c), (f1, c1))):
        several, one = microseconds(lambda: op(top, *args, nv)), microseconds(lambda: op(top, *alone))
        print(f"Q{k} {op.__name__}: {nv} vectors {several:.1f} us, one {one:.1f} us", flush=True)
        assert several <= nv * one
