"""An adjoint whose waits give up: no wait may be taken for a result, neither by the launches
queued behind it nor by a later call."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu
ETIMEOUT = -4


def _backward_fails(s):
    s.set_option(M.OPT_SPIN_LIMIT, 1)  # (from the host: every wait gives up at once and every kernel ends)
    with pytest.raises(M.MplpError) as e:
        s.adjoint_backward()
    assert e.value.code == ETIMEOUT
    s.set_option(M.OPT_SPIN_LIMIT, 0)


# one-workgroup forwards keep no records: every segment's are made by the backward, the last
# one's shorter than the buffer, in tiles of 16 and 32 labels and with the records of one
# segment only
@pytest.mark.parametrize("n,L,K,every", [(8, 4, 7, 3), (5, 27, 11, 4), (8, 16, 3, 5)])
def test_segments_behind_a_failed_recomputation(n, L, K, every):
    print("CASE", n, L, K, every, flush=True)
    model = W.uniform(n, L, seed=n + L, dtype=np.float64)
    with M.Solver.from_model(model) as s, M.Solver.from_model(model) as ref:
        ref.adjoint_forward(K, every)
        want = ref.adjoint_backward()
        s.adjoint_forward(K, every)
        _backward_fails(s)
        for x, y in zip(s.adjoint_backward(), want):
            assert np.array_equal(x, y)


# finite costs whose sums overflow: no argmin may leave the labels.  Whatever labels the
# records name, an update's reverse keeps the sum of its two nodes' adjoints (rows and
# columns of the table included), so the unary gradient sums to the number of nodes that
# seeded it (one each; a node whose values are all NaN may or may not).
@pytest.mark.parametrize("n,L", [(8, 7), (40, 20), (40, 33), (30, 64)])
def test_records_name_labels_whatever_overflows(n, L):
    print("CASE", n, L, flush=True)
    model = W.uniform(n, L, seed=L, dtype=np.float64)
    rng = np.random.default_rng(n)
    model.unaries[:] = 1e308 * rng.uniform(-1, 1, model.unaries.shape)
    model.pairwise[:] = 1.7e308 * rng.uniform(-1, 1, model.pairwise.shape)
    with M.Solver.from_model(model) as s:
        s.adjoint_forward(5, 2)
        U = s.get_state()[0]
        gu, gp = s.adjoint_backward()
        again = s.adjoint_backward()
    assert np.isfinite(gu).all() and np.isfinite(gp).all()
    seeds = round(float(gu.sum()))
    assert (U < np.inf).any(1).sum() <= seeds <= n
    assert abs(gu.sum() - seeds) <= 1e-12 * gu.size * max(1.0, np.abs(gu).max())
    assert np.array_equal(gu, again[0]) and np.array_equal(gp, again[1])


# a backward that fails, or one on the other engine, has overwritten what the forward
# recorded: the next one starts from the checkpoints
@pytest.mark.parametrize("K,every", [(3, 3), (6, 3), (8, 3), (9, 2)])
def test_backward_after_a_failed_one(K, every):
    print("CASE", K, every, flush=True)
    model = W.uniform(40, 20, seed=K, dtype=np.float64)
    with M.Solver.from_model(model) as s, M.Solver.from_model(model) as ref:
        ref.adjoint_forward(K, every)
        want = ref.adjoint_backward()
        s.adjoint_forward(K, every)
        _backward_fails(s)
        for x, y in zip(s.adjoint_backward(), want):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("K,every", [(3, 3), (6, 3), (8, 3), (9, 2)])
def test_backward_on_both_engines(K, every):
    print("CASE", K, every, flush=True)
    model = W.uniform(40, 20, seed=K, dtype=np.float64)
    with M.Solver.from_model(model) as s:
        s.adjoint_forward(K, every)
        got = []
        for engine in (M.ENGINE_STEP, 0, M.ENGINE_STEP, 0, 0):
            s.set_option(M.OPT_ENGINE, engine)
            got.append(s.adjoint_backward())
    for g in got[1:]:
        assert np.array_equal(g[0], got[0][0]) and np.array_equal(g[1], got[0][1])
