"""lbm_workspace_size at the largest checkpoint intervals: with one segment the
size is linear in the interval (every area of the record is whole 256 bytes)."""

import numpy as np
import pytest

from paper_2402_10809_amd import lbm

INT_MAX = 2 ** 31 - 1


@pytest.mark.parametrize("T", [1, 5])
@pytest.mark.parametrize("ckpt", [INT_MAX, INT_MAX - 1, INT_MAX - 2, INT_MAX - 3, 10 ** 9])
def test_one_segment_of_any_length(T, ckpt):
    g = lbm.lbm_grid()
    g.nx, g.ny, g.nz = 8, 6, 5
    solid = np.zeros((5, 6, 8), np.uint8)
    size = [lbm.lbm_workspace_size(g, solid, T, c) for c in (10, 11)]
    assert lbm.lbm_workspace_size(g, solid, T, ckpt) == size[0] + (size[1] - size[0]) * (ckpt - 10)
