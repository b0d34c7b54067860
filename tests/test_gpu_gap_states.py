"""iterate_gap's bounds and labellings from copies of the messages, taken many iterations
at a time, against iterate(1), dual_bound and decode in turn: every tile of the launch
that keeps the copies, and the models that copy after each launch."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu

MODELS = [
    ("ragged 16", lambda: W.uniform(30, 13, seed=1), 7, {}),
    ("full 16", lambda: W.uniform(31, 16, seed=2), 2, {}),
    ("ragged 32", lambda: W.uniform(24, 17, seed=3), 5, {}),
    ("full 32", lambda: W.uniform(60, 32, seed=4), 6, {}),
    ("ragged 64", lambda: W.uniform(21, 45, seed=5), 4, {}),
    ("full 64", lambda: W.uniform(40, 64, seed=6), 3, {}),
    ("above 64", lambda: W.uniform(14, 70, seed=7), 3, {}),
    ("one workgroup", lambda: W.uniform(6, 4, seed=8), 9, {}),
    ("one iteration", lambda: W.uniform(25, 9, seed=9), 1, {}),
    ("FP64", lambda: W.uniform(20, 12, seed=10, dtype=np.float64), 4, {}),
    ("two at a time", lambda: W.uniform(260, 55, seed=11), 5, {}),
    ("one at a time", lambda: W.uniform(330, 60, seed=12), 2, {}),
    ("step engine", lambda: W.uniform(20, 12, seed=13), 4, {M.OPT_ENGINE: M.ENGINE_STEP}),
    ("update (M)", lambda: W.uniform(20, 12, seed=14), 4, {M.OPT_RULE: M.RULE_M}),
    ("few slots a workgroup", lambda: W.chain(41, 20, seed=15), 4, {}),
]


@pytest.mark.parametrize("name,make,k,options", MODELS, ids=[m[0] for m in MODELS])
def test_states_are_those_of_single_iterations(name, make, k, options):
    model = make()
    with M.Solver.from_model(model) as s, M.Solver.from_model(model) as t:
        for key, value in options.items():
            s.set_option(key, value)
            t.set_option(key, value)
        s.iterate(1)
        t.iterate(1)
        for _ in range(2):  # (the second call in the first one's workspace)
            dual, energy, labels = s.iterate_gap(k)
            want = []
            for _ in range(k):
                t.iterate(1)
                want.append((t.dual_bound(), *t.decode()))
            assert [float(x) for x in dual] == [w[0] for w in want]
            assert [float(x) for x in energy] == [w[2] for w in want]
            best = int(np.argmin([w[2] for w in want]))
            assert np.array_equal(labels, want[best][1])
        for x, y in zip(s.get_state(), t.get_state()):
            assert np.asarray(x).tobytes() == np.asarray(y).tobytes()
