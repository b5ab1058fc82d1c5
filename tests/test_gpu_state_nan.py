"""lbm_get_state returns what the state holds: only the unknowns beyond an open
face read as 0; a diverged state's values that are not numbers come back so."""

import numpy as np
import pytest

from paper_2402_10809_amd import Solver
from synth import as_d3q27, tiny_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("q27", [False, True])
@pytest.mark.parametrize("kind", ["open", "open_extrap", "periodic"])
@pytest.mark.parametrize("steps", [2, 3])
def test_nan_round_trip(kind, steps, q27, storage):
    case = tiny_case(kind, seed=2)
    case = as_d3q27(case) if q27 else case
    s = Solver.from_case(case, storage=storage)
    s.step(steps)
    f, om = s.get_state()
    print(f"NaN round trip {kind} steps={steps} q27={q27} {storage}", flush=True)
    assert np.all(np.isfinite(f))
    x = s.fluid_index() % case.nx
    inner = np.flatnonzero((x > 1) & (x < case.nx - 2))
    bad = np.zeros(f.shape, bool)
    rng = np.random.default_rng(5)
    bad[rng.integers(0, f.shape[0], 40), rng.choice(inner, 40)] = True
    g = f.copy()
    g[bad] = np.nan
    s.set_state(g, om)
    h, om2 = s.get_state()
    assert np.array_equal(np.isnan(h), bad)
    assert np.array_equal(om, om2)
    assert np.abs(h[~bad] - f[~bad]).max() <= 2.0 ** -51
