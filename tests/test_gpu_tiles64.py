"""FP64 around the tile of 48 labels and the adjoint's records at 64, bit for bit against
the per-matching engine: both edges of the tile, messages in LDS and in memory,
workgroups that own one, two and more slots."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu

MODELS = [
    ("33 labels", lambda: W.uniform(12, 33, seed=1, dtype=np.float64)),
    ("47 labels", lambda: W.uniform(11, 47, seed=2, dtype=np.float64)),
    ("48 labels", lambda: W.uniform(12, 48, seed=3, dtype=np.float64)),
    ("49 labels", lambda: W.uniform(11, 49, seed=4, dtype=np.float64)),
    ("64 labels", lambda: W.uniform(13, 64, seed=5, dtype=np.float64)),
    ("one slot each, 40", lambda: W.chain(9, 40, seed=6)),
    ("one slot each, 64", lambda: W.chain(9, 64, seed=7)),
    ("messages in memory", lambda: W.uniform(230, 40, seed=8, dtype=np.float64)),
]


@pytest.mark.parametrize("name,make", MODELS, ids=[m[0] for m in MODELS])
def test_forward_and_adjoint_are_the_step_engine(name, make):
    model, got = make(), []
    for engine in (M.ENGINE_PERSISTENT, M.ENGINE_STEP):
        with M.Solver.from_model(model) as s:
            s.set_option(M.OPT_ENGINE, engine)
            s.iterate(2)
            out = [s.iterate_trace(2), *s.get_state()]
            out += [np.float64(s.adjoint_forward(5, 2)), *s.adjoint_backward(), *s.get_state()]
            got.append(out)
    for x, y in zip(*got):
        x, y = np.ascontiguousarray(x), np.ascontiguousarray(y)
        assert x.dtype == y.dtype and x.tobytes() == y.tobytes()
