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
