"""The outputs and transfers of a state at the edges of their launches: dense fields
(every voxel written, whatever the alignment and the set of planes), FP64
diagnostics around one workgroup's run of cells, the state in fluid order through
the stage area, and the reverse of more velocity iterates than are kept.
"""

import ctypes as ct

import numpy as np
import pytest
import torch

import oracle
from paper_2402_10809_amd import Solver, lbm
from synth import aniso_shape, as_d3q27, make_config, periodic_box_case, tiny_case, tiny_random

pytestmark = pytest.mark.gpu

FIELDS = (("rho", 1), ("u", 3), ("shear", 1), ("omega", 1), ("sigma", 6), ("tau", 3))


def _fields(s, names, shift=0):
    """lbm_moments into NaN-filled buffers that start `shift` floats off 256 bytes."""
    bufs = {}
    for n, k in FIELDS:
        if n in names:
            raw = torch.full((k * s.nbox + shift,), float("nan"), device="cuda")
            bufs[n] = raw[shift:].view(k, s.nbox)
    ptr = [ct.c_void_p(bufs[n].data_ptr()) if n in bufs else None for n, _ in FIELDS]
    lbm.check(lbm.lib().lbm_moments(s.ctx, *ptr))
    return {n: b.cpu().numpy() for n, b in bufs.items()}


@pytest.mark.parametrize("q27", [False, True])
@pytest.mark.parametrize("seed", range(6))
def test_dense_fields_write_every_voxel(seed, q27):
    case = tiny_random(seed)
    s = Solver.from_case(as_d3q27(case) if q27 else case)
    s.step(3 + seed % 2)
    print(f"dense fields {case.nx}x{case.ny}x{case.nz} q27={q27}", flush=True)
    full = _fields(s, [n for n, _ in FIELDS])
    fluid = case.solid.reshape(-1) == 0
    assert np.all(full["rho"][0, fluid] > 0.5)
    for n, a in full.items():
        assert np.all(np.isfinite(a)), n
        assert np.all(a[:, ~fluid] == 0), n
    for names, shift in ((["rho"], 0), (["u", "tau"], 1), (["sigma", "omega"], 2)):
        part = _fields(s, names, shift)
        for n in names:
            assert np.array_equal(part[n], full[n]), (n, shift)


def test_dense_fields_beyond_the_cache_are_the_same():
    """512x320x320: one plane (210 MB) is written in one launch, several are cleared first."""
    s = Solver.from_case(make_config("c2"))
    s.step(5)
    one, two = _fields(s, ["omega"]), _fields(s, ["omega", "shear"])
    assert np.array_equal(one["omega"], two["omega"])
    assert np.all(np.isfinite(two["shear"]))


@pytest.mark.parametrize("shape", [(16, 16, 1), (64, 64, 64), (64, 64, 65), (91, 67, 88)])
def test_diagnostics_around_the_run_length(shape):
    """256, 262 144 (one block of cells per workgroup at most), 266 240 and 536 536
    cells.  The sums of n FP64 terms of one sign are within n 2^-53 of each other
    in any order; the velocity and omega compared are rounded to FP32."""
    nx, ny, nz = shape
    case = periodic_box_case(nx=nx, ny=ny, nz=nz, ell=3.0, g=1e-4)
    s = Solver.from_case(case)
    s.step(7)
    d = s.diagnostics()
    f, _ = s.get_state()
    m = s.moments()
    n = s.n_fluid
    print(f"diagnostics of {n} cells: mass {d['mass']:.12e} max|u| {d['max_u']:.6e}", flush=True)
    assert n == nx * ny * nz and d["nonfinite"] == 0
    assert abs(d["mass"] - f.sum()) <= 20 * n * 2.0 ** -53 * f.sum()
    u = m["u"].double()
    assert abs(d["max_u"] - float(u.pow(2).sum(0).sqrt().max())) <= 2.0 ** -22 * d["max_u"]
    om = m["omega"].double()
    assert abs(d["min_omega"] - float(om.min())) <= 2.0 ** -23 and abs(d["max_omega"] - float(om.max())) <= 2.0 ** -23
    ke = float((0.5 * m["rho"].double() * u.pow(2).sum(0)).sum())
    assert abs(d["ke"] - ke) <= 2.0 ** -20 * ke


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("q27", [False, True])
@pytest.mark.parametrize("seed", range(4))
def test_state_round_trip(seed, q27, storage):
    """f = v / U + rest rounds v / U to 2^-53 of the O(1) rest value, so a second
    solver's populations come back within 2^-51 with FP32 storage; with FP16 the
    value that comes back is the stored one unless it lies within that of zero."""
    case = tiny_random(seed)
    case = as_d3q27(case) if q27 else case
    a, b = Solver.from_case(case, storage=storage), Solver.from_case(case, storage=storage)
    steps = 4 + seed % 2
    a.step(steps)
    b.step(steps % 2)
    f, om = a.get_state()
    print(f"state {case.nx}x{case.ny}x{case.nz} q27={q27} {storage}: {a.n_fluid} cells", flush=True)
    b.set_state(f=f)
    b.set_state(omega=om)
    f2, om2 = b.get_state()
    assert np.array_equal(om, om2)
    assert np.abs(f2 - f).max() <= 2.0 ** -51
    assert a.n_fluid == int((case.solid == 0).sum())


def test_state_through_large_buffers():
    """A state of 28 MB, whose pages are touched by several threads first."""
    case = periodic_box_case(nx=64, ny=48, nz=60, ell=4.0)
    s = Solver.from_case(case)
    s.step(2)
    f, om = s.get_state()
    again = np.full_like(f, np.nan)
    o2 = np.full_like(om, np.nan)
    lbm.check(lbm.lib().lbm_get_state(s.ctx, again.ctypes.data_as(ct.c_void_p), o2.ctypes.data_as(ct.c_void_p)))
    assert f.nbytes > 8 << 20
    assert np.array_equal(f, again) and np.array_equal(om, o2)


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("iters", [1, 2, 10, 11, 13])
def test_reverse_of_the_velocity_iterates(iters, fp64):
    """The first ten iterates' norms are kept, later ones are computed again."""
    case = tiny_case("open", seed=1)
    case.wave = (0.1, 0.5, 20.0)
    case.porous = dict(case.porous, forchheimer=1, d=0.5, aniso=aniso_shape(), aniso_iters=iters)
    T, tb, te, ck = 12, 4, 12, 5
    J_ref, g_ref = oracle.Oracle(case).grad_reverse(T, tb, te, ck, "ke")
    s = Solver.from_case(case, adjoint_T=T, ckpt=ck)
    J, g = s.adjoint(tb, te, T, ck, fp64=fp64)
    fluid = case.solid == 0
    err = np.abs(g.cpu().numpy() - g_ref)[fluid].max() / np.abs(g_ref)[fluid].max()
    print(f"iterates {iters} fp64={fp64}: J {J:.10e} oracle {J_ref:.10e}, gradient max-rel {err:.3e}", flush=True)
    assert abs(J - J_ref) <= 1e-5 * abs(J_ref)
    assert err < 1e-4
