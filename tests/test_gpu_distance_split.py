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
