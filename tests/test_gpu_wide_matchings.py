"""Matchings with more edges than compute units on the tiles of 80, 96 and 112 labels, and a
grid whose mapped launch would not fit the chip: bit for bit the per-matching engine."""
import numpy as np
import pytest

import paper_2004_08227_amd as M
from paper_2004_08227_amd import workloads as W

pytestmark = pytest.mark.gpu


def _same(model, grid):
    got = []
    for engine in (M.ENGINE_PERSISTENT, M.ENGINE_STEP):
        with M.Solver.from_model(model) as s:
            s.set_option(M.OPT_ENGINE, engine)
            if engine == M.ENGINE_PERSISTENT:
                s.set_option(M.OPT_GRID, grid)
                print("CASE", model.n, model.L, model.m, "grid", s.info("grid"), flush=True)
            s.iterate(3)
            got.append(s.get_state(comp=True))
    for x, y in zip(*got):
        assert x.tobytes() == y.tobytes()


@pytest.mark.parametrize("L", [65, 80, 96, 100, 112])
def test_more_edges_than_compute_units(L):
    n, rng = 620, np.random.default_rng(L)
    ring = np.array([(u, u + 1) for u in range(n - 1)] + [(0, n - 1)], dtype=np.int32)
    model = W.Model(n, L, ring, rng.random((n, L), dtype=np.float32), rng.random((n, L, L), dtype=np.float32))
    _same(model, 0)


def test_mapped_launch_beyond_the_chip():
    _same(W.uniform(162, 6, seed=1), 243)  # 81 positions, three workgroups each: 264 mapped


@pytest.mark.parametrize("L,threads", [(13, 256), (16, 256), (13, 64), (20, 64), (29, 256)])
def test_traces_at_the_largest_grid(L, threads):
    """The largest grid that is accepted, and the default of a matching that fills it, fit the
    chip in every kernel that may run there; traces need more registers than iterations."""
    m, rng = 1500, np.random.default_rng(L)
    pairs = rng.permutation(2 * m).reshape(m, 2)
    edges = np.concatenate([pairs, np.stack([pairs[:-1, 0], pairs[1:, 1]], 1)]).astype(np.int32)
    n = 2 * m
    model = W.Model(n, L, edges, rng.random((n, L), dtype=np.float32), rng.random((len(edges), L, L), dtype=np.float32))
    most, got = 0, []
    for grid in (None, 0):
        with M.Solver.from_model(model) as s:
            s.set_option(M.OPT_THREADS, threads)
            s.set_option(M.OPT_SPIN_LIMIT, 1 << 20)
            if grid is None:
                for per_cu in range(1, 17):
                    try:
                        s.set_option(M.OPT_GRID, 256 * per_cu)
                        most = 256 * per_cu
                    except M.MplpError:
                        break
            assert s.info("grid") <= most
            print("CASE", L, threads, "grid", s.info("grid"), "largest", most, flush=True)
            t = s.iterate_trace(3)
            s.iterate(2)
            for rule in (M.RULE_M, M.RULE_U):
                if threads == 256:
                    s.set_option(M.OPT_RULE, rule)
                    s.iterate(2)
            got.append([t, *s.get_state(comp=True)])
    with M.Solver.from_model(model) as s:
        s.set_option(M.OPT_ENGINE, M.ENGINE_STEP)
        s.iterate_trace(3)
        s.iterate(2)
        for rule in (M.RULE_M, M.RULE_U):
            if threads == 256:
                s.set_option(M.OPT_RULE, rule)
                s.iterate(2)
        want = s.get_state(comp=True)
    for g in got:
        assert np.array_equal(g[0], got[0][0])
        for x, y in zip(g[1:], want):
            assert x.tobytes() == y.tobytes()
    if (L, threads) == (13, 256):  # 67 registers: seven waves a SIMD, two of them of every workgroup
        assert most == 3 * 256


@pytest.mark.parametrize("kind", [M.COST_POTTS, M.COST_TRUNC_LINEAR, M.COST_TRUNC_QUAD])
def test_structured_costs_in_label_order(kind):
    """700 edges a matching on one compute wave in label order: the quadratic kind's kernel has
    room for two workgroups on a compute unit, the others' for eight."""
    n, L, rng = 1400, 9, np.random.default_rng(kind)
    ring = np.array([(u, u + 1) for u in range(n - 1)] + [(0, n - 1)], dtype=np.int32)
    prm = rng.random((n, M.COST_PARAMS[kind]), dtype=np.float32)
    if kind != M.COST_POTTS:
        prm[:, 1] = rng.integers(1, 2 * L, n)
    model, got = W.Model(n, L, ring, rng.random((n, L), dtype=np.float32), prm), []
    for threads in (64, 256):
        with M.Solver.from_structured(model, kind) as s:
            s.set_option(M.OPT_THREADS, threads)
            print("CASE", kind, threads, "grid", s.info("grid"), flush=True)
            s.iterate(3)
            got.append((*s.get_state(comp=True), s.dual_bound()))
    if kind == M.COST_TRUNC_LINEAR:  # (other sums: FP32 rounding of costs up to 1 a few updates long)
        assert np.abs(got[0][0] - got[1][0]).max() <= 1e-5
    else:
        assert all(np.array_equal(x, y) for x, y in zip(*got))


OPTIONS = [
    ("threads after the grid", 13, [(M.OPT_THREADS, 64), (M.OPT_GRID, 1280), (M.OPT_THREADS, 256)]),
    ("(M), then the grid", 48, [(M.OPT_RULE, M.RULE_M), (M.OPT_GRID, 512)]),
    ("(U), then the grid", 17, [(M.OPT_RULE, M.RULE_U), (M.OPT_GRID, 700)]),
    ("(M), large tile", 113, [(M.OPT_RULE, M.RULE_M), (M.OPT_GRID, 300)]),
    ("per matching, then the grid", 40, [(M.OPT_ENGINE, M.ENGINE_STEP), (M.OPT_GRID, 512), (M.OPT_ENGINE, 0)]),
]


@pytest.mark.parametrize("name,L,options", OPTIONS, ids=[o[0] for o in OPTIONS])
def test_grids_set_under_other_options(name, L, options):
    m, rng = (1300, np.random.default_rng(L)) if L <= 64 else (400, np.random.default_rng(L))
    edges = rng.permutation(2 * m).reshape(m, 2).astype(np.int32)
    model = W.Model(2 * m, L, edges, rng.random((2 * m, L), dtype=np.float32), rng.random((m, L, L), dtype=np.float32))
    got = []
    for engine in (None, M.ENGINE_STEP):
        with M.Solver.from_model(model) as s:
            s.set_option(M.OPT_SPIN_LIMIT, 1 << 20)
            for key, value in options:
                try:
                    s.set_option(key, value)
                except M.MplpError:  # (a limit of these options: nothing larger runs then)
                    assert key == M.OPT_GRID
            if engine is not None:
                s.set_option(M.OPT_ENGINE, engine)
            print("CASE", name, s.info("grid"), flush=True)
            s.iterate(3)
            got.append(s.get_state(comp=True))
    for x, y in zip(*got):
        assert x.tobytes() == y.tobytes()
