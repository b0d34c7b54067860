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
