"""The FP32 mailbox engine bit for bit against the per-matching one on its tiles of 80, 96
and 112 labels and at their edges, with messages in LDS and in memory, prefetched and not
(few and many slots a workgroup), and at ragged counts below (whole rows are read)."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu


def run(model, opts):
    with M.Solver.from_model(model) as s:
        for k, v in opts.items():
            s.set_option(k, v)
        s.iterate(3)
        return list(s.get_state(comp=True)) + [np.float64(s.dual_bound())]


@pytest.mark.parametrize("L", [17, 31, 33, 63, 64, 65, 79, 80, 81, 95, 96, 97, 111, 112, 113, 127, 128])
@pytest.mark.parametrize("n,density", [(7, 1.0), (22, 1.0), (30, 0.1)], ids=["few", "many", "one each"])
def test_tiles_are_the_step_engine(L, n, density):
    model = W.random_graph_model(n, L, density, seed=L * n, dtype=np.float32)
    ref = run(model, {M.OPT_ENGINE: M.ENGINE_STEP})
    for phi in (1, 2):
        got = run(model, {M.OPT_ENGINE: M.ENGINE_PERSISTENT, M.OPT_PHI: phi})
        for a, b in zip(got, ref):
            assert a.tobytes() == b.tobytes()


@pytest.mark.parametrize("L", [40, 70, 90, 110])
def test_tiles_large_costs(L):
    model = W.random_graph_model(10, L, 1.0, seed=L, dtype=np.float32, lo=-1.0)
    model.pairwise *= np.float32(9e17)
    a = run(model, {M.OPT_ENGINE: M.ENGINE_PERSISTENT})
    b = run(model, {M.OPT_ENGINE: M.ENGINE_STEP})
    assert all(x.tobytes() == y.tobytes() for x, y in zip(a, b))
