"""The one-workgroup engine of small models: bit for bit the per-matching engine, state,
trace, dual and rounding, at the edges of its tiles (1, 7..9, 15..17, 31, 32 labels) and
of its range of matchings (one edge to one wave per edge and beyond), and across a change
of engine in the middle of a run."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu


def star(n, L, dtype):
    m = W.random_graph_model(n, L, 1.0, seed=n, dtype=dtype)
    keep = m.edges[:, 0] == 0
    return W.Model(n, L, m.edges[keep], m.unaries, np.ascontiguousarray(m.pairwise[keep]), "star")


def run(model, engine, splits):
    with M.Solver.from_model(model) as s:
        s.set_option(M.OPT_ENGINE, engine)
        out = []
        for k, trace in splits:
            if trace:
                out.append(s.iterate_trace(k))
            else:
                s.iterate(k)
        return out + list(s.get_state(comp=True)) + [np.float64(s.dual_bound()), s.decode()[0]]


def same(a, b):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        x, y = np.ascontiguousarray(x), np.ascontiguousarray(y)
        assert x.dtype == y.dtype and x.tobytes() == y.tobytes()


SHAPES = [(2, 1), (2, 8), (3, 2), (5, 7), (8, 4), (9, 9), (16, 15), (17, 16), (12, 17), (16, 24), (20, 8), (24, 31), (25, 32),
          (31, 5), (32, 16), (33, 8), (34, 8)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,L", SHAPES)
def test_solo_is_the_step_engine(n, L, dtype):
    model = W.uniform(n, L, seed=7 * n + L, dtype=dtype)
    splits = [(1, False), (3, True), (2, False), (1, True)]
    same(run(model, M.ENGINE_AUTO, splits), run(model, M.ENGINE_STEP, splits))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("name", ["star", "chain", "sparse", "ties"])
def test_solo_graphs(name, dtype):
    if name == "star":
        model = star(60, 11, dtype)
    elif name == "chain":
        model = W.chain(26, 13, seed=3).astype(dtype)
    else:
        model = W.random_graph_model(40, 6, 0.15, seed=5, dtype=dtype)
        if name == "ties":
            rng = np.random.default_rng(1)
            model.unaries[:] = rng.integers(0, 3, model.unaries.shape)
            model.pairwise[:] = rng.integers(-2, 3, model.pairwise.shape)
    splits = [(4, True), (3, False)]
    same(run(model, M.ENGINE_AUTO, splits), run(model, M.ENGINE_STEP, splits))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_solo_large_costs_and_engine_change(dtype):
    model = W.uniform(14, 10, seed=2, dtype=dtype)
    model.pairwise *= dtype(1e17 if dtype == np.float32 else 1e290)
    ref = run(model, M.ENGINE_STEP, [(5, False)])
    same(run(model, M.ENGINE_AUTO, [(5, False)]), ref)
    with M.Solver.from_model(model) as s:
        s.iterate(2)
        s.set_option(M.OPT_ENGINE, M.ENGINE_PERSISTENT)
        s.iterate(2)
        s.set_option(M.OPT_ENGINE, M.ENGINE_AUTO)
        s.iterate(1)
        same(list(s.get_state(comp=True)), ref[:3])


def test_solo_noalloc_and_adjoint():
    """The no-allocation call and the FP64 forward of the adjoint take the same engine."""
    import torch
    model = W.uniform(18, 11, seed=4)
    un, pw = torch.from_numpy(model.unaries).cuda(), torch.from_numpy(model.pairwise).cuda()
    U, phi = torch.empty_like(un), torch.empty((model.m, 2, model.L), device="cuda")
    d = M.solve_noalloc(model.edges, un, pw, 6, U, phi)
    with M.Solver.from_model(model) as s:
        s.set_option(M.OPT_ENGINE, M.ENGINE_STEP)
        s.iterate(6)
        Us, ps = s.get_state()
        same([U.cpu().numpy(), phi.cpu().numpy(), np.float64(d)], [Us, ps, np.float64(s.dual_bound())])
    got = []
    for engine in (M.ENGINE_AUTO, M.ENGINE_STEP):
        with M.Solver.from_model(model) as s:
            s.set_option(M.OPT_ENGINE, engine)
            loss = s.adjoint_forward(7, 3)
            got.append([np.float64(loss), *s.adjoint_backward(), *s.get_state(comp=True)])
    same(got[0], got[1])
