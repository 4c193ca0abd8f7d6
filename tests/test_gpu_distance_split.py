"""Whole runs against the oracle at populations around the column blocks of the
distances: those among P_t start beside the searches in whole blocks of 128
columns, the rest follows them."""

import numpy as np
import pytest

from paper_2103_10453_amd import instances as gen
from paper_2103_10453_amd import plse as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("p,depth", [
    (63, 120), (64, 120), (65, 120), (127, 120), (128, 120), (129, 120), (200, 120), (257, 60),
    (4097, 12), (4225, 12),  # units of 16 rows
])
def test_solve_around_column_blocks(torch_cuda, oracle_mod, p, depth):
    print(f"[gpu-case] distance split p={p}", flush=True)
    g = gen.random_greedy(14, 0.5, 23)
    s = P.Solver(g, depth=depth)
    grid, filled = s.solve(p, 3, 9000 + p)
    st = s.stats()
    I = oracle_mod.Instance(g)
    r = I.run(I.params(depth=depth), p, 3, 9000 + p)
    assert filled == r["filled"]
    np.testing.assert_array_equal(grid, r["grid"])
    np.testing.assert_array_equal(st["best_f_per_gen"], r["best_f"][:r["gens"]])
    np.testing.assert_array_equal(st["counters_per_gen"], r["counters"][:r["gens"]])


def test_batch_with_distances_of_both_kinds(torch_cuda):
    """A batch of several search groups whose distances start in two parts
    equals the instances solved alone."""
    print("[gpu-case] batch of 5 instances p=130 G=2", flush=True)
    grids = [gen.random_greedy(12, 0.6, 5), gen.random_greedy(20, 0.5, 7),
             gen.planted(33, 0.45, 9), gen.random_greedy(45, 0.7, 4), gen.planted(10, 0.4, 0)]
    p, seeds = 130, [3, 1, 4, 1, 5]
    kw = [dict(depth=300, variant=int(k == 1)) for k in range(5)]
    solvers = [P.Solver(g, **k) for g, k in zip(grids, kw)]
    res = P.Solver.solve_batch(solvers, p, 2, seeds)
    for g, k, s, seed, (grid, filled) in zip(grids, kw, solvers, seeds, res):
        alone = P.Solver(g, **k)
        want, f = alone.solve(p, 2, seed)
        assert f == filled
        np.testing.assert_array_equal(grid, want)
        np.testing.assert_array_equal(s.stats()["counters_per_gen"],
                                      alone.stats()["counters_per_gen"])
