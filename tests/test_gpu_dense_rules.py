"""lbm_moments on either side of its rules (zeros in the same launch or cleared
first; the rows in XCD shares or in launch order): the same fields whatever set
of buffers is asked for, and the density that the populations give."""

import ctypes as ct

import numpy as np
import pytest
import torch

from paper_2402_10809_amd import Solver, lbm
from synth import aneurysm_case, as_d3q27, periodic_box_case

pytestmark = pytest.mark.gpu

PLANES = dict(rho=1, u=3, shear=1, omega=1, sigma=6, tau=3)


def _fields(s, names):
    bufs = {n: torch.full((k, s.nbox), float("nan"), device="cuda") for n, k in PLANES.items() if n in names}
    lbm.check(lbm.lib().lbm_moments(s.ctx, *[ct.c_void_p(bufs[n].data_ptr()) if n in bufs else None for n in PLANES]))
    return {n: b.cpu().numpy() for n, b in bufs.items()}


@pytest.mark.parametrize("nx", [64, 66, 65])
def test_fields_do_not_depend_on_the_buffers_asked_for(nx):
    """nx % 4 zero and not, planes on 16 bytes and not; one plane, several planes of
    one buffer, two, three and six buffers."""
    case = aneurysm_case(nx, 31, 29, R=5, Rs=7, ell=3, seed=4)
    s = Solver.from_case(case)
    s.step(9)
    print(f"dense rules {nx}x31x29", flush=True)
    full = _fields(s, list(PLANES))
    solid = case.solid.reshape(-1) != 0
    for n, a in full.items():
        assert np.all(np.isfinite(a)) and np.all(a[:, solid] == 0), n
    for names in (["rho"], ["tau"], ["sigma"], ["u", "omega"], ["rho", "shear"], ["rho", "u", "omega"]):
        part = _fields(s, names)
        for n in names:
            assert np.array_equal(part[n], full[n]), names


@pytest.mark.parametrize("q27", [False, True])
def test_fields_of_a_state_beyond_the_cache(q27):
    """3.28 M cells (302 MB of state on D3Q19): density against the
    populations, rho being FP32 (2^-24 of itself, and the FP32 sums of
    q populations behind them)."""
    case = periodic_box_case(nx=128, ny=160, nz=160, ell=6.0, g=1e-4)
    case = as_d3q27(case) if q27 else case
    s = Solver.from_case(case)
    s.step(3)
    print(f"dense fields of {s.n_fluid} cells, q27={q27}", flush=True)
    m = _fields(s, ["rho", "u"])
    f, _ = s.get_state()
    rho = f.sum(0) / case.phi.reshape(-1)
    q = f.shape[0]
    assert np.abs(m["rho"][0] - rho).max() <= q * 2.0 ** -24 * rho.max()
    assert np.all(np.isfinite(m["u"])) and m["u"][0].mean() > 0
