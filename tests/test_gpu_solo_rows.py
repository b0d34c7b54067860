"""The one-workgroup engine whose lanes read rows and columns of labels: every label count
of its tiles, one matching per iteration, idle waves, and models that fill its LDS, bit
for bit against the per-matching engine."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu


def star(n, L, dtype, seed):
    rng = np.random.default_rng(seed)
    edges = np.stack([np.zeros(n - 1, np.int32), np.arange(1, n, dtype=np.int32)], 1)
    return W.Model(n, L, edges, rng.random((n, L)).astype(dtype), rng.random((n - 1, L, L)).astype(dtype), f"star{n}")


MODELS = [(f"{np.dtype(d).name} L={L}", lambda d=d, L=L: W.uniform(7, L, seed=L, dtype=d))
          for d, labels in ((np.float32, range(1, 9)), (np.float64, list(range(1, 18)) + [23, 24, 25, 31, 32])) for L in labels]
MODELS += [
    ("one matching", lambda: W.uniform(2, 8, seed=1)),
    ("one matching FP64", lambda: W.uniform(2, 13, seed=2, dtype=np.float64)),
    ("two matchings", lambda: W.chain(5, 8, seed=3)),
    ("idle waves", lambda: W.random_graph_model(20, 7, 0.3, seed=4)),
    ("LDS full", lambda: star(1084, 8, np.float32, 5)),
    ("LDS full FP64", lambda: star(498, 12, np.float64, 6)),
    ("12 edges FP64", lambda: W.uniform(24, 16, seed=7, dtype=np.float64)),
]


@pytest.mark.parametrize("name,make", MODELS, ids=[m[0] for m in MODELS])
def test_is_the_step_engine(name, make):
    model, got = make(), []
    for engine in (M.ENGINE_AUTO, M.ENGINE_STEP):
        with M.Solver.from_model(model) as s:
            s.set_option(M.OPT_ENGINE, engine)
            s.iterate(3)
            out = [s.iterate_trace(2)] if model.unaries.dtype == np.float64 else []
            s.iterate(2)
            got.append(out + list(s.get_state()))
    for x, y in zip(*got):
        x, y = np.ascontiguousarray(x), np.ascontiguousarray(y)
        assert x.dtype == y.dtype and x.tobytes() == y.tobytes()
