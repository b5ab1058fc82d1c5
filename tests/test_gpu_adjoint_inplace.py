"""The reverse sweep's in-place adjoint populations against the FP64 oracle: first
reverse steps of both parities (T odd and even, down to one step), every
segment length around them, FP32 and FP64 populations.

Bound on an entry's error: the gradient tolerance of the adjoint, 1e-4 of the
largest entry, plus what FP32 storage leaves of an entry that cancels to zero.
After one step the gradient does vanish (the oracle holds 1e-20 of it), so only
the second term bounds it there: an entry is sum_i w_i a_i over the stored
adjoints a_i, each rounded to 2^-24 of itself a step, and with the region mean
of rho |u|^2 / 2 as objective |a_i| is at most |c_i| |u| / N + |u|^2 / 2N <= 2 |u| / N
on a region of N cells, |u| <= sqrt(2 J N).
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
    region = int((case.sac & fluid).sum())
    scale = np.abs(g_ref)[fluid].max()
    err = np.abs(g.cpu().numpy() - g_ref)[fluid].max()
    stored = T * 2.0 ** -24 * 2.0 * np.sqrt(2.0 * J_ref / region)
    print(f"  J {J:.10e} oracle {J_ref:.10e}; gradient error {err:.3e} of {scale:.3e}, storage {stored:.3e}", flush=True)
    assert abs(J - J_ref) <= 1e-5 * abs(J_ref) + 1e-30
    assert err < 1e-4 * scale + stored


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("kind", ["open", "open_extrap", "periodic"])
@pytest.mark.parametrize("T", [7, 8, 9, 12])
def test_segments_recorded_while_the_next_is_reversed(T, kind, fp64):
    """Segment lengths around T: a last segment of one step, short and full ones,
    one segment only.  The recorded trajectory is the same in every case, so the
    gradients are the same bits as with the whole record."""
    case = tiny_case(kind, seed=5)
    if kind == "periodic":
        case.porous = dict(case.porous, g=tuple(50.0 * v for v in case.porous["g"]))
    else:
        case.wave = (0.04, 0.5, 20.0)
    s = Solver.from_case(case, adjoint_T=T, ckpt=T)
    J, g = s.adjoint(T // 3, T, T, T, fp64=fp64)
    for ckpt in (1, 2, 3, 4, T - 1, T + 3):
        print(f"segments {kind} T={T} ckpt={ckpt} fp64={fp64}", flush=True)
        s2 = Solver.from_case(case, adjoint_T=T, ckpt=ckpt)
        J2, g2 = s2.adjoint(T // 3, T, T, ckpt, fp64=fp64)
        assert J2 == J
        assert np.array_equal(g2.cpu().numpy(), g.cpu().numpy())
