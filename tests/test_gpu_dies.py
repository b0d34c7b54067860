"""The map of workgroups to positions of a matching: every logical workgroup once for
every size (host), and models at its edges bit for bit against the per-matching engine."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

DIES = 8


def logical(G, ms, b):
    d, die, i = G // ms, b % DIES, b // DIES
    p = die * ms // DIES + i // d
    return i % d * ms + p if p < (die + 1) * ms // DIES else G


@pytest.mark.parametrize("ms", list(range(8, 129)))
def test_every_workgroup_once(ms):
    for d in (1, 2, 3, 4):
        G, launch = ms * d, DIES * (-(-ms // DIES)) * d
        got = [logical(G, ms, b) for b in range(launch)]
        assert sorted(w for w in got if w < G) == list(range(G))
        assert all(w <= G for w in got)


MODELS = [
    ("7 positions", lambda: W.uniform(14, 20, seed=1)),
    ("8 positions", lambda: W.uniform(16, 20, seed=2)),
    ("9 positions", lambda: W.uniform(18, 33, seed=3)),
    ("30 positions, odd nodes", lambda: W.uniform(61, 21, seed=4)),
    ("unequal matchings", lambda: W.random_graph_model(60, 20, 0.5, seed=5)),
    ("more than 256 workgroups", lambda: W.uniform(250, 4, seed=6)),
    ("tile of 80", lambda: W.uniform(20, 70, seed=7)),
]


@pytest.mark.gpu
@pytest.mark.parametrize("name,make", MODELS, ids=[m[0] for m in MODELS])
def test_is_the_step_engine(name, make):
    model, got = make(), []
    for engine in (M.ENGINE_PERSISTENT, M.ENGINE_STEP):
        with M.Solver.from_model(model) as s:
            s.set_option(M.OPT_ENGINE, engine)
            s.iterate(3)
            got.append([s.iterate_trace(2), *s.get_state()])
    assert np.allclose(got[0][0], got[1][0], rtol=1e-6, atol=0)
    for x, y in zip(got[0][1:], got[1][1:]):
        assert np.asarray(x).tobytes() == np.asarray(y).tobytes()


@pytest.mark.gpu
@pytest.mark.parametrize("n,L", [(24, 17), (40, 40)])
def test_structured_costs(n, L):
    rng = np.random.default_rng(n)
    edges = np.array([(u, v) for u in range(n) for v in range(u + 1, n)], dtype=np.int32)
    un, w = rng.random((n, L)).astype(np.float32), rng.random(len(edges)).astype(np.float32)
    table = np.where(np.eye(L, dtype=bool), np.float32(0), w[:, None, None]).astype(np.float32)
    with M.Solver.from_potts(W.Model(n, L, edges, un, w)) as a, M.Solver(n, L, edges, un, table) as b:
        b.set_option(M.OPT_ENGINE, M.ENGINE_STEP)
        a.iterate(3)
        b.iterate(3)
        for x, y in zip(a.get_state(), b.get_state()):
            assert np.asarray(x).tobytes() == np.asarray(y).tobytes()
