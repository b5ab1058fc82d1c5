"""Contexts coming and going beside other work on the GPU: destroying one makes no
device call, and more contexts may be alive than there are slots of pinned memory
for their reductions' results."""

import numpy as np
import pytest
import torch

from paper_2402_10809_amd import Solver
from synth import as_d3q27, tiny_case

pytestmark = pytest.mark.gpu


def test_destroy_does_not_wait_for_other_streams():
    s = Solver.from_case(tiny_case("open", seed=0))
    s.step(2)
    s.diagnostics()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    print("close a context beside a stream with 0.1 s of work", flush=True)
    with torch.cuda.stream(side):
        torch.cuda._sleep(200_000_000)
        done = torch.cuda.Event()
        done.record()
    s.close()
    running = not done.query()
    torch.cuda.synchronize()
    assert running


def test_destroy_beside_a_capture():
    s = Solver.from_case(tiny_case("open", seed=0))
    x = torch.zeros(1000, device="cuda")
    torch.cuda.synchronize()
    print("close a context while a graph is captured", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        x += 1
        s.close()
        x += 2
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert float(x[0]) == float(x[-1]) == 3.0 * (k + 1)


@pytest.mark.parametrize("q27", [False, True])
def test_more_contexts_than_slots(q27):
    """70 contexts alive at once (64 slots), then their slots in use again."""
    case = tiny_case("open", seed=1)
    case = as_d3q27(case) if q27 else case
    for turn in range(2):
        print(f"70 contexts, turn {turn}, q27={q27}", flush=True)
        many = [Solver.from_case(case) for _ in range(70)]
        for k, s in enumerate(many):
            s.step(5 + k % 3)
        got = [list(s.diagnostics().values()) for s in many]
        noalloc = [list(s.diagnostics_noalloc().values()) for s in many]
        for k in range(70):
            assert np.array_equal(got[k], got[k % 3]) and np.array_equal(noalloc[k], got[k]), k
        assert got[0][10] == 5 and got[1][0] != got[0][0]
        for s in many[::2]:
            s.close()
        again = Solver.from_case(case)
        again.step(5)
        assert list(again.diagnostics().values()) == got[0]
