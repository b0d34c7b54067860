"""Every tile of the wave engine (multiples of 8 labels, both edges of each) bit for bit
against single handles: models on one workgroup in LDS, on one workgroup through the
mailboxes, and on teams."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu

LABELS = [3, 8, 9, 16, 17, 23, 24, 25, 32, 33, 39, 40, 41, 48, 49, 55, 56, 57, 63, 64]


@pytest.mark.parametrize("n,labels,options", [
    (9, LABELS, {}),
    (9, LABELS, {"lds": 0}),
    (31, [17, 24, 33, 40], {}),
    (30, [41, 48, 49, 56], {}),
    (33, [57, 64, 25, 32], {"grid": 64}),
    (3, [39, 40, 47, 55], {"lds": 0}),
], ids=["lds", "mailboxes", "teams to 40", "teams to 56", "teams to 64", "one slot a worker"])
def test_batches_are_single_handles(n, labels, options):
    models = [W.uniform(n, L, seed=100 * n + L) for L in labels]
    with M.Batch(models) as b:
        for key, value in options.items():
            b.set_option(key, value)
        b.set_option("engine", 2)
        b.iterate(3)
        b.iterate(2)
        states = [b.get_state(i) for i in range(len(models))]
    for model, state in zip(models, states):
        with M.Solver.from_model(model) as s:
            s.iterate(5)
            for x, y in zip(state, s.get_state()):
                assert np.asarray(x).tobytes() == np.asarray(y).tobytes()
