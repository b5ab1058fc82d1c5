"""lbm_adjoint on the launch forms that small lattices do not reach: whole waves
of interior cells (which step through their wave records), workgroups of four
waves (from 262 144 compact cells on), and segments recorded and reversed in
turn (above 786 432), against the FP64 oracle's reverse sweep and across
segment lengths.

Bound on a gradient entry's error: 1e-4 of the largest entry, the gradient
tolerance of the adjoint, plus what FP32 storage leaves of an entry whose terms
cancel.  An entry is sum_i w_i a_i over the adjoints a_i of the populations, which
carry a relative error of 2^-24 per step (their own storage, or with FP64 ones
that of the recorded state they are linear in).  On a region of N cells the
objectives give |a_i| <= |c_i| |u| / N + |u|^2 / 2N <= 2 |u| / N (kinetic energy) and
|a_i| <= |c_i|^2 |1 - omega / 2| / N <= 2 / N (wall shear stress).  With FP64 adjoint
populations and the kinetic energy, where nothing cancels, only the recorded
state is rounded: an entry is a sum of products of at most four of its values a
step, so 4 T 2^-24 of the largest entry (populations rounded to FP32 miss that).
"""

import numpy as np
import pytest

import oracle
from paper_2402_10809_amd import Solver
from synth import Case, aneurysm_case, aniso_shape, tiny_case

pytestmark = pytest.mark.gpu


def _duct(nx, ny, nz, seed=0, aniso=False, outlet=1):
    """An open duct, walls in y, periodic in z, driven by its inflow and a body
    force: pure fluid, then porosity 0.8, then random porosity along x, with
    solid voxels in one half of it only."""
    rng = np.random.default_rng(seed)
    solid = (rng.random((nz, ny, nx)) < 0.01).astype(np.uint8)
    solid[nz // 2:] = 0
    solid[:, :, 0] = solid[:, :, nx - 1] = 0
    phi = np.ones((nz, ny, nx), np.float32)
    phi[:, :, nx // 3: 2 * nx // 3] = 0.8
    phi[:, :, 2 * nx // 3: nx - 3] = rng.uniform(0.7, 0.9, (nz, ny, nx - 3 - 2 * nx // 3))
    phi[solid != 0] = 0.0
    porous = dict(nu_d=0.1, kc=180.0, d=2.0, forchheimer=0, g=(1e-3, 4e-4, -3e-4))
    if aniso:
        porous.update(forchheimer=1, d=0.5, aniso=aniso_shape(seed), aniso_iters=6)
    return Case(name=f"duct{nx}x{ny}x{nz}", nx=nx, ny=ny, nz=nz, periodic=(False, False, True), solid=solid, phi=phi,
                sac=(rng.random((nz, ny, nx)) < 0.5) & (solid == 0), inlet=True, outlet=outlet,
                inlet_shape=rng.uniform(0.2, 1.0, (nz, ny)).astype(np.float32), wave=(0.04, 0.5, 20.0), porous=porous)


def _against_oracle(case, T, tb, kind, fp64, J, g):
    o = oracle.Oracle(case)
    J_ref, g_ref = o.grad_reverse(T, tb, T, T, kind)
    f, om = o.init()
    o.run(f, om, 0, T - 1)
    m = o.moments(f, om, T - 1)
    region = case.sac.reshape(-1)[o.cells()]
    if kind == "wss":
        region = region & (np.abs(m["tau"]).sum(0) > 0)
        a = 2.0
    else:
        a = 2.0 * np.sqrt((m["u"] ** 2).sum(0).max())
    fluid = case.solid == 0
    scale = np.abs(g_ref)[fluid].max()
    err = np.abs(g - g_ref)[fluid].max()
    bound = 1e-4 * scale + T * 2.0 ** -24 * a / region.sum()
    if fp64 and kind == "ke":
        bound = 4 * T * 2.0 ** -24 * scale
    print(f"  J {J:.10e} oracle {J_ref:.10e}; gradient error {err:.3e} of {scale:.3e}, bound {bound:.3e}", flush=True)
    assert abs(J - J_ref) <= 1e-5 * abs(J_ref)
    assert err < bound
    assert np.all(g[~fluid] == 0)


@pytest.mark.parametrize("kind,fp64,aniso,outlet", [("ke", False, False, 1), ("ke", True, False, 2),
                                                    ("wss", False, True, 2), ("wss", True, True, 1)])
@pytest.mark.parametrize("shape", [(200, 44, 32), (280, 56, 51)])
def test_large_grids(shape, kind, fp64, aniso, outlet):
    """281 600 and 799 680 compact cells: four waves to a workgroup, segments
    recorded in the reverse launches and in turn."""
    case = _duct(*shape, seed=1, aniso=aniso, outlet=outlet)
    T, tb = 6, 1
    got = []
    for ckpt in (2, 1, 4, T):
        print(f"large adjoint {case.name} {kind} fp64={fp64} aniso={aniso} ckpt={ckpt}", flush=True)
        s = Solver.from_case(case, adjoint_T=T, ckpt=ckpt)
        J, g = s.adjoint(tb, T, T, ckpt, kind=kind, fp64=fp64)
        got.append((J, g.cpu().numpy()))
        s.close()
    _against_oracle(case, T, tb, kind, fp64, *got[0])
    for J, g in got[1:]:
        assert J == got[0][0]
        assert np.array_equal(g, got[0][1])


@pytest.mark.parametrize("kind", ["ke", "wss"])
@pytest.mark.parametrize("name", ["bulk", "vessel", "duct", "duct_aniso"])
def test_segments_with_whole_interior_waves(name, kind):
    """Objective windows over several segments, on lattices with waves of 64
    interior cells: the gradient is the same bits whatever the segment length."""
    if name == "bulk":
        case = tiny_case("bulk", seed=2)
    elif name == "vessel":
        case = aneurysm_case(160, 32, 32, R=6, Rs=9, ell=3, seed=4, wave=(0.05, 0.5, 200.0))
    else:
        case = _duct(150, 14, 12, seed=3, aniso=name == "duct_aniso")
    case.porous = dict(case.porous, g=(1e-3, 4e-4, -3e-4))
    for T, tb in ((24, 5), (9, 0)):
        s = Solver.from_case(case, adjoint_T=T, ckpt=T)
        J, g = s.adjoint(tb, T, T, T, kind=kind)
        g = g.cpu().numpy()
        for ckpt in (1, 2, 3, 7, T - 1):
            s2 = Solver.from_case(case, adjoint_T=T, ckpt=ckpt)
            J2, g2 = s2.adjoint(tb, T, T, ckpt, kind=kind)
            g2 = g2.cpu().numpy()
            print(f"segments {name} {kind} T={T} ckpt={ckpt}: J off by {abs(J2 - J) / abs(J):.1e}, gradient by "
                  f"{np.abs(g2 - g).max() / np.abs(g).max():.1e}, entries {np.count_nonzero(g2 != g)}", flush=True)
            assert J2 == J
            assert np.array_equal(g2, g)
