"""The reverse sweep's in-place adjoint populations against the FP64 oracle: first
reverse steps of both parities (T odd and even, down to one step), every
segment length around them, FP32 and FP64 populations.  Bound: the gradient
tolerance of the adjoint, 1e-4 of the largest entry (FP32 populations: 19
roundings of 2^-24 a step, below 1e-5 over five steps).
"""

import numpy as np
import pytest

import oracle
from paper_2402_10809_amd import Solver
from synth import tiny_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("T,ckpt", [(1, 1), (2, 1), (2, 5), (4, 3), (5, 1), (5, 2), (5, 5)])
@pytest.mark.parametrize("kind", ["open", "open_extrap", "periodic"])
def test_short_reverse_sweeps(kind, T, ckpt, fp64):
    case = tiny_case(kind, seed=3)
    if kind == "periodic":
        case.porous = dict(case.porous, g=tuple(50.0 * v for v in case.porous["g"]))
    else:
        case.wave = (0.04, 0.5, 20.0)
    print(f"reverse sweep {kind} T={T} ckpt={ckpt} fp64={fp64}", flush=True)
    J_ref, g_ref = oracle.Oracle(case).grad_reverse(T, 0, T, ckpt, "ke")
    s = Solver.from_case(case, adjoint_T=T, ckpt=ckpt)
    J, g = s.adjoint(0, T, T, ckpt, kind="ke", fp64=fp64)
    fluid = case.solid == 0
    scale = np.abs(g_ref)[fluid].max()
    err = np.abs(g.cpu().numpy() - g_ref)[fluid].max() / max(scale, 1e-300)
    print(f"  J {J:.10e} oracle {J_ref:.10e}; gradient max-rel {err:.3e} of {scale:.3e}", flush=True)
    assert abs(J - J_ref) <= 1e-5 * abs(J_ref) + 1e-30
    assert err < 1e-4 or scale < 1e-20
