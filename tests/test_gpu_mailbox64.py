"""The FP64 mailbox engine bit for bit against the per-matching one where its ways change:
ragged tiles of two words a label, workgroups that own one slot, messages too many for LDS,
traces, and the adjoint with records from the forward and from recomputation, backward
called twice."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu


def same(a, b):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        x, y = np.ascontiguousarray(x), np.ascontiguousarray(y)
        assert x.dtype == y.dtype and x.tobytes() == y.tobytes()


def forward(model, engine):
    with M.Solver.from_model(model) as s:
        s.set_option(M.OPT_ENGINE, engine)
        s.iterate(2)
        tr = s.iterate_trace(2)
        s.iterate(1)
        return [tr, *s.get_state(), np.float64(s.dual_bound()), s.decode()[0]]


MODELS = [
    ("ragged tile 16", lambda: W.uniform(35, 13, seed=1, dtype=np.float64)),
    ("ragged tile 32", lambda: W.uniform(36, 31, seed=2, dtype=np.float64)),
    ("full tile 32", lambda: W.uniform(37, 32, seed=3, dtype=np.float64)),
    ("tile 64 from 33", lambda: W.uniform(12, 33, seed=4, dtype=np.float64)),
    ("ragged tile 64", lambda: W.uniform(20, 63, seed=5, dtype=np.float64)),
    ("full tile 64", lambda: W.uniform(10, 64, seed=6, dtype=np.float64)),
    ("one slot each", lambda: W.chain(41, 20, seed=7)),
    ("greedy", lambda: W.random_graph_model(90, 9, 0.2, seed=8)),
    ("messages in memory", lambda: W.uniform(1300, 2, seed=9, dtype=np.float64)),
]


@pytest.mark.parametrize("name,make", MODELS, ids=[m[0] for m in MODELS])
def test_forward_is_the_step_engine(name, make):
    model = make()
    same(forward(model, M.ENGINE_PERSISTENT), forward(model, M.ENGINE_STEP))


@pytest.mark.parametrize("name,make,K,every", [
    ("one segment", MODELS[0][1], 3, 5), ("two", MODELS[1][1], 4, 2), ("three", MODELS[3][1], 5, 2), ("five", MODELS[4][1], 9, 2),
    ("one slot each", MODELS[6][1], 7, 3), ("greedy", MODELS[7][1], 5, 1), ("one workgroup", lambda: W.uniform(14, 7, seed=3), 6, 2),
], ids=lambda v: v if isinstance(v, str) else None)
def test_adjoint_twice_is_the_step_engine(name, make, K, every):
    model, got = make(), []
    for engine in (M.ENGINE_AUTO, M.ENGINE_STEP):
        with M.Solver.from_model(model) as s:
            s.set_option(M.OPT_ENGINE, engine)
            loss = s.adjoint_forward(K, every)
            first = s.adjoint_backward()
            got.append([np.float64(loss), *first, *s.adjoint_backward(), *s.get_state()])
    same(got[0], got[1])
    same(got[0][1:3], got[0][3:5])
