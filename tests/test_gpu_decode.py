"""GPU rounding (Eq. (5)) and its energy (Eq. (1)), label for label and bit for bit
against a plain numpy walk of the nodes in the library's summation order, at the sizes
where the kernel changes its ways: degrees around a block of incidences, tables at the
limit of the LDS copy, label counts around one and two per lane, sparse graphs and nodes
without edges."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu


def walk(model, phi, order):
    """Nodes ascending; incidence k of a node (in slot order) belongs to partial sum k mod
    16, which adds the message into the node and, for an edge to a lower node v, the
    reparametrized row of v's label; the 16 partial sums are added to the unary in order;
    ties go to the smallest label.  FP64 throughout."""
    un, pw = model.unaries.astype(np.float64), model.pairwise.astype(np.float64)
    phi = phi.astype(np.float64)
    inc = [[] for _ in range(model.n)]
    for e in order.tolist():
        inc[model.edges[e, 0]].append((e, 0))
        inc[model.edges[e, 1]].append((e, 1))
    x = np.zeros(model.n, np.int64)
    for u in range(model.n):
        part = np.zeros((16, model.L))
        for k, (e, side) in enumerate(inc[u]):
            part[k % 16] += phi[e, side]
            if side:
                y = x[model.edges[e, 0]]
                part[k % 16] += pw[e, y] - phi[e, 0, y] - phi[e, 1]
        c = un[u].copy()
        for p in part:
            c += p
        x[u] = int(c.argmin())
    terms = [un[np.arange(model.n), x], pw[order, x[model.edges[order, 0]], x[model.edges[order, 1]]]]
    # the sum of the energy: 1024 strided partial sums, then halves
    acc = np.zeros(1024)
    for t in terms:
        for i in range(0, t.size, 1024):
            acc[:t[i:i + 1024].size] += t[i:i + 1024]
    while acc.size > 1:
        acc = acc[:acc.size // 2] + acc[acc.size // 2:]
    return x, acc[0]


CASES = [
    ("one node", np.float32, 1, 3, 1.0), ("no edges", np.float32, 5, 7, 0.0), ("one label", np.float32, 9, 1, 1.0),
    ("one block", np.float32, 257, 5, 1.0), ("block edge", np.float32, 258, 3, 1.0), ("three blocks", np.float32, 600, 2, 1.0),
    ("sparse", np.float32, 300, 16, 0.03), ("full wave", np.float32, 33, 64, 1.0), ("two a lane", np.float32, 33, 65, 1.0),
    ("copied", np.float32, 20, 106, 1.0), ("too large", np.float32, 20, 107, 1.0), ("largest", np.float32, 12, 128, 1.0),
    ("two a lane, blocks", np.float32, 140, 66, 1.0), ("double", np.float64, 130, 6, 1.0), ("double full", np.float64, 20, 64, 1.0),
    ("double two a lane", np.float64, 70, 65, 1.0), ("double largest", np.float64, 9, 128, 1.0),
]


@pytest.mark.parametrize("name,dtype,n,L,density", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("whole", [False, True], ids=["real", "ties"])
def test_decode_walk(name, dtype, n, L, density, whole):
    model = W.random_graph_model(n, L, density, seed=n + L, dtype=dtype)
    if whole:  # integer costs from the start: many exact ties
        rng = np.random.default_rng(n * L)
        model.unaries[:] = rng.integers(0, 3, model.unaries.shape)
        model.pairwise[:] = rng.integers(0, 3, model.pairwise.shape)
    with M.Solver.from_model(model) as s:
        for k in (0, 3):
            s.iterate(k)
            labels, energy = s.decode()
            ref, ref_energy = walk(model, s.get_state()[1], s.schedule()[1])
            np.testing.assert_array_equal(labels, ref)
            assert energy == ref_energy


@pytest.mark.parametrize("kind", [M.COST_POTTS, M.COST_TRUNC_LINEAR, M.COST_TRUNC_QUAD])
def test_decode_structured(kind):
    make = {M.COST_POTTS: W.potts_pure, M.COST_TRUNC_LINEAR: W.trunc_linear, M.COST_TRUNC_QUAD: W.trunc_quad}[kind]
    prm, dense = make(40, 21, 0.6, seed=3)
    with M.Solver.from_structured(prm, kind) as s:
        s.iterate(4)
        labels, energy = s.decode()
        ref, ref_energy = walk(dense, s.get_state()[1], s.schedule()[1])
    np.testing.assert_array_equal(labels, ref)
    assert energy == ref_energy


@pytest.mark.parametrize("n,L,dtype", [(3, 1, np.float32), (40, 20, np.float64), (131, 16, np.float32), (101, 13, np.float64),
                                       (230, 5, np.float32), (90, 100, np.float32), (70, 3, np.float64)])
def test_dual_bound_and_state_order(n, L, dtype):
    """The bound recomputed in numpy from the state the call returns, whose messages are in
    the caller's edge order (ordered on the host below 1 MB, on the device from there on),
    with edges given in a shuffled order and both orientations."""
    model = W.random_graph_model(n, L, 0.9, seed=n, dtype=dtype)
    rng = np.random.default_rng(L)
    order = rng.permutation(model.m)
    e, pw = model.edges[order].copy(), model.pairwise[order].copy()
    flip = rng.random(model.m) < 0.5
    e[flip] = e[flip][:, ::-1]
    pw[flip] = pw[flip].transpose(0, 2, 1)
    with M.Solver(n, L, e, model.unaries, pw) as s:
        s.iterate(2)
        d = s.dual_bound()
        U, phi, c = s.get_state(comp=True)
    lo, hi = e.min(1), e.max(1)
    th = np.where(flip[:, None, None], pw.transpose(0, 2, 1), pw).astype(np.float64)
    node = model.unaries.astype(np.float64).copy()
    np.add.at(node, lo, phi[:, 0].astype(np.float64))
    np.add.at(node, hi, phi[:, 1].astype(np.float64))
    assert np.abs(node - (U.astype(np.float64) + c)).max() <= (1e-4 if dtype == np.float32 else 1e-11)
    edge = (th - phi[:, 0].astype(np.float64)[:, :, None] - phi[:, 1].astype(np.float64)[:, None, :]).reshape(len(e), -1).min(1)
    ref = node.min(1).sum() + edge.sum()
    assert abs(d - ref) <= 1e-12 * max(1.0, abs(ref)) * model.m
