"""bench.py's flops per pass against the axes that each form of the three passes
transforms, counted here one transform at a time (5 N log2 of its points)."""
import math
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402

# axes transformed in the plane, pencil and accumulate pass
AXES = {"line": ((1,), (2, 3, 3, 2), (1,)), "register": ((2, 3), (1, 1), (3, 2)), "slab": ((2, 3), (1, 1, 3), (2,))}


@pytest.mark.parametrize("grid,s,form", [((32, 32, 32), 8, "slab"), ((72, 72, 72), 8, "slab"), ((60, 60, 60), 8, "register"),
                                         ((24, 72, 72), 8, "register"), ((24, 24, 60), 8, "line"), ((32, 32, 32), 16, "line"),
                                         ((36, 40, 45), 16, "line"), ((45, 45, 45), 8, "line")])
def test_passes_are_rated_by_their_own_axes(grid, s, form):
    assert bench.three_pass_form(grid, s) == form
    n = grid[0] * grid[1] * grid[2]
    m = bench.kernel_model(grid, s)
    for kind, axes, rest in zip(("plane", "pencil", "accumulate"), AXES[form], (6, 2, 8)):
        want = sum(5 * n * math.log2(grid[a - 1]) for a in axes) + rest * n
        assert m[kind]["flops"] == pytest.approx(want, rel=1e-12)
    e_axes = ((1,), (2, 3)) if form == "line" and s == 16 else ((2, 3), (1,))
    for kind, axes, rest in zip(("energy_plane", "energy_pencil"), e_axes, (6, 3)):
        want = sum(5 * n * math.log2(grid[a - 1]) for a in axes) + rest * n
        assert m[kind]["flops"] == pytest.approx(want, rel=1e-12)
