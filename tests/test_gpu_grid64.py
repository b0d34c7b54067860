"""MPLPXX_OPT_GRID on the FP64 mailbox engine: used, reported and without effect on results;
the values that were accepted and refused before."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,per_cu", [(9, 7), (24, 7), (50, 4)])
def test_any_grid(L, per_cu):
    model, want = W.uniform(40, L, seed=L, dtype=np.float64), None
    for grid in (0, 1, 3, 20, 41, 256, 257, 256 * per_cu):
        print("CASE", L, grid, flush=True)
        with M.Solver.from_model(model) as s:
            s.set_option(M.OPT_GRID, grid)
            assert s.info("grid") == (40 if grid == 0 else min(grid, 256))
            s.iterate(2)
            got = [s.iterate_trace(3), *s.get_state()]
            with pytest.raises(M.MplpError):
                s.set_option(M.OPT_GRID, 256 * per_cu + 1)
        want = want or got
        assert all(np.array_equal(x, y) for x, y in zip(got, want))
