"""The limit for the waits of iterations does not end a rounding, whose nodes wait for their
labels in turn."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limit", [1, 1000])
@pytest.mark.parametrize("n,L,dtype", [(300, 16, np.float32), (600, 2, np.float64), (70, 65, np.float32)])
def test_decode_under_any_limit(n, L, dtype, limit):
    print("CASE", n, L, limit, flush=True)
    model = W.uniform(n, L, seed=n, dtype=dtype)
    with M.Solver.from_model(model) as s:
        s.iterate(2)
        want, energy = s.decode()
        s.set_option(M.OPT_SPIN_LIMIT, limit)
        got, e = s.decode()
    assert np.array_equal(got, want) and e == energy
