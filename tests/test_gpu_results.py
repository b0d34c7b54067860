"""Results that fit the handle's pinned memory and results that do not (traces, labels,
states below, at and above its 64 KiB): the same values either way."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 8183, 8184, 8185])  # 64 KiB - 64 bytes are 8184 doubles
def test_traces(k):
    model = W.uniform(4, 3, seed=1)
    with M.Solver.from_model(model) as a, M.Solver.from_model(model) as b:
        got = a.iterate_trace(k)
        want = np.concatenate([b.iterate_trace(min(1000, k - i)) for i in range(0, k, 1000)])
        assert np.asarray(got).tobytes() == want.tobytes()


@pytest.mark.parametrize("n", [16368, 16369])  # 64 KiB - 64 bytes are 16368 labels
def test_labels(n):
    rng = np.random.default_rng(n)
    un = rng.random((n, 3)).astype(np.float32)
    edges = np.array([[0, n - 1]], dtype=np.int32)
    pw = rng.random((1, 3, 3)).astype(np.float32)
    with M.Solver(n, 3, edges, un, pw) as s:
        labels, energy = s.decode()
    want = un.argmin(1)
    assert np.array_equal(labels[1:-1], want[1:-1])
    x = labels.astype(np.int64)
    assert abs(energy - (un.astype(np.float64)[np.arange(n), x].sum() + float(pw[0, x[0], x[-1]]))) < 1e-9 * n


@pytest.mark.parametrize("n,L,dtype", [(33, 13, np.float32), (34, 14, np.float32), (12, 60, np.float64), (13, 60, np.float64), (1, 5, np.float32)])
def test_states(n, L, dtype):
    model = W.uniform(n, L, seed=n, dtype=dtype)
    with M.Solver.from_model(model) as s, M.Solver.from_model(model) as t:
        s.iterate(3)
        U, phi = s.get_state()[:2]
        t.set_state(U, phi)
        assert t.dual_bound() == s.dual_bound()
        for x, y in zip(t.get_state()[:2], (U, phi)):
            assert np.asarray(x).tobytes() == np.asarray(y).tobytes()
        assert np.asarray(s.get_state()[0]).tobytes() == np.asarray(U).tobytes()
