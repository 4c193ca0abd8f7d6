"""Population update (Alg. 4) with the candidates' places in LDS and in the
workspace, the key order in global memory both times, against the oracle."""

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


@pytest.mark.parametrize("p,hook", [(8193, 0), (8193, 1), (2049, 1), (3000, 1)])
def test_select_places(torch_cuda, oracle_mod, p, hook):
    """Families of near copies, some larger than a close list holds."""
    torch = torch_cuda
    print(f"[gpu-case] select places p={p} hook={hook}", flush=True)
    g = gen.random_greedy(12, 0.6, 7)
    s = P.Solver(g, select_global_sort=hook)
    nv, m = s.nv, 2 * p
    rng = np.random.default_rng(p)
    X = rng.integers(0, 6, size=(m, s.stride), dtype=np.uint8)
    X[:, nv:] = 0
    X[rng.integers(0, m, size=m // 2)] = X[rng.integers(0, m, size=m // 2)]
    big = rng.choice(m, size=120, replace=False)
    X[big] = X[big[0]]
    X[big, rng.integers(0, nv, size=120)] = 7
    D = s.stage_distances(torch.from_numpy(X).cuda())
    f = rng.integers(0, 3, size=m).astype(np.int32)
    acc = s.stage_select(torch.from_numpy(f).cuda(), D, 3, 77)
    torch.cuda.synchronize()
    want = oracle_mod.select(nv, p, 10, 77, 3, f, D.cpu().numpy().astype(np.int32))
    np.testing.assert_array_equal(acc.cpu().numpy(), want)


@pytest.mark.parametrize("shift", [0, 1, 3, 7])
@pytest.mark.parametrize("p", [100, 2052])
def test_select_shifted_rows(torch_cuda, oracle_mod, p, shift):
    """A matrix of distances at any two-byte address, with close lists longer
    than are kept, whose rows the selection reads itself."""
    torch = torch_cuda
    print(f"[gpu-case] select shifted p={p} shift={shift}", flush=True)
    s = P.Solver(gen.random_greedy(12, 0.6, 7))
    nv, m = s.nv, 2 * p
    rng = np.random.default_rng(p + shift)
    group = rng.integers(0, m // 50, size=m)  # about fifty close to each other
    D = np.where(group[:, None] == group[None, :], 1, nv).astype(np.int16)
    np.fill_diagonal(D, 0)
    buf = torch.zeros(m * m + 8, dtype=torch.int16, device="cuda")
    Dg = buf[shift:shift + m * m].view(m, m)
    Dg.copy_(torch.from_numpy(D))
    f = rng.integers(0, 3, size=m).astype(np.int32)
    acc = s.stage_select(torch.from_numpy(f).cuda(), Dg, 3, 77)
    torch.cuda.synchronize()
    want = oracle_mod.select(nv, p, 10, 77, 3, f, D.astype(np.int32))
    np.testing.assert_array_equal(acc.cpu().numpy(), want)


def _chain(m, width):
    """Candidates in key order (f ascending), each close to the next `width`."""
    D = np.full((m, m), 50, dtype=np.int16)
    for k in range(1, width + 1):
        i = np.arange(m - k)
        D[i, i + k] = D[i + k, i] = 3
    np.fill_diagonal(D, 0)
    return D


@pytest.mark.parametrize("p,width,step,hook", [
    (5, 1, 1, 0), (12, 1, 1, 0), (16, 13, 1, 0), (32, 1, 1, 0),   # six rounds and fewer
    (33, 2, 1, 0), (100, 13, 1, 0), (700, 1, 1, 0), (1500, 5, 3, 0),
    (1500, 16, 1, 0),                                             # lists of 32, all that are kept
    (1500, 20, 1, 0),                                             # longer ones between them
    (2100, 1, 1, 1), (2100, 7, 40, 1),
])
def test_select_chains(torch_cuda, oracle_mod, p, width, step, hook):
    """Chains of close candidates as long as the population, in key order or
    (steps of f) broken by the draws."""
    torch = torch_cuda
    print(f"[gpu-case] select chain p={p} width={width} step={step} hook={hook}", flush=True)
    s = P.Solver(gen.random_greedy(12, 0.6, 7), select_global_sort=hook)
    m = 2 * p
    D = _chain(m, width)
    f = (np.arange(m) // step).astype(np.int32)
    acc = s.stage_select(torch.from_numpy(f).cuda(), torch.from_numpy(D).cuda(), 3, 77)
    torch.cuda.synchronize()
    want = oracle_mod.select(s.nv, p, 10, 77, 3, f, D.astype(np.int32))
    np.testing.assert_array_equal(acc.cpu().numpy(), want)


def test_select_chain_time(torch_cuda):
    """One wave decides 64 candidates in 6 us: 128 times that for 8192 in one
    chain, six times the selection of candidates far apart (128 us); twice
    that is allowed.  Rounds as long as the chain took 34 times."""
    torch = torch_cuda
    p = 4096
    s = P.Solver(gen.random_greedy(16, 0.4, 5))
    s.ensure_workspace(p)
    f = torch.arange(2 * p, dtype=torch.int32, device="cuda")
    acc = torch.zeros(p, dtype=torch.int32, device="cuda")
    us = {}
    for name, width in (("apart", 0), ("chain", 1)):
        D = torch.from_numpy(_chain(2 * p, width)).cuda()
        best = float("inf")
        for _ in range(8):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            P.plse_stage_select(s.h, p, 2, 9, f, D, acc)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        us[name] = 1e3 * best
    print(f"[gpu-case] select apart {us['apart']:.0f} us, chain {us['chain']:.0f} us", flush=True)
    assert us["chain"] < 12 * us["apart"]
