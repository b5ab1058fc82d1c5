"""Calls that a program may capture into a HIP graph, replayed several times with
its own work between the replays: every replay gives what the call itself gives."""

import ctypes as ct

import numpy as np
import pytest
import torch

from paper_2402_10809_amd import Solver, lbm
from synth import as_d3q27, make_config, tiny_case

pytestmark = pytest.mark.gpu

PLANES = dict(rho=1, u=3, shear=1, omega=1, sigma=6, tau=3)


def _solver(case, stream, **kw):
    with torch.cuda.stream(stream):
        return Solver.from_case(case, stream=stream, **kw)


def _moments(s, bufs):
    lbm.check(lbm.lib().lbm_moments(s.ctx, *[ct.c_void_p(bufs[n].data_ptr()) if n in bufs else None for n in PLANES]))


@pytest.mark.parametrize("names", [["rho"], ["u", "rho"], list(PLANES)])
@pytest.mark.parametrize("name", ["tiny", "tiny_q27", "c1", "c2"])
def test_moments_under_capture(name, names):
    """Outputs in one launch and cleared first (one plane, more than 256 MB)."""
    if name == "c2" and len(names) == len(PLANES):
        names = ["u", "tau"]
    case = tiny_case("open", seed=4) if name.startswith("tiny") else make_config(name)
    case = as_d3q27(case) if name.endswith("q27") else case
    stream = torch.cuda.Stream()
    s = _solver(case, stream)
    s.step(3)
    bufs = {n: torch.empty((PLANES[n], s.nbox), device="cuda") for n in names}
    print(f"moments under capture: {name} {names}", flush=True)
    torch.cuda.synchronize()
    _moments(s, bufs)
    torch.cuda.synchronize()
    want = {n: b.clone() for n, b in bufs.items()}
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        _moments(s, bufs)
    for k in range(4):
        for b in bufs.values():
            b.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for n in names:
            assert torch.equal(bufs[n], want[n]), (n, k)


@pytest.mark.parametrize("q27", [False, True])
@pytest.mark.parametrize("kind", ["open", "open_extrap"])
def test_reset_and_steps_under_capture(kind, q27):
    """Six steps from rest, captured with the reset before them: each replay ends at
    the same state, whatever was stepped in between."""
    case = tiny_case(kind, seed=3)
    case = as_d3q27(case) if q27 else case
    stream = torch.cuda.Stream()
    s = _solver(case, stream)
    print(f"reset and steps under capture: {kind} q27={q27}", flush=True)
    s.reset()
    s.step(6)
    f, om = s.get_state()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        s.reset()
        s.step(6)
    for k in range(4):
        s.step(2 * k)  # an even number: the context's time counts on from the captured steps
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        g, om2 = s.get_state()
        assert np.array_equal(f, g) and np.array_equal(om, om2), k
