"""Shared-space block CG at the edges of its m x m steps (block sizes around the 8-row and 16-column
tiles, the largest block, dependent and zero columns), against the oracle's run of the method:
the first iterates agree to 1e-12 per column and the ranks after deflation are the true ones
(a converged solve of consistent dependent columns)."""
import numpy as np
import pytest

import oracle
from paper_2509_17257_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 7, 8, 9, 15, 17, 33, 48, 63, 64])
def test_first_iterates(m):
    import paper_2509_17257_amd as h2x
    P = W.sphere_points(2500, 600)
    prm = dict(ell=0.5, shift=1.0, eta=1.0, leaf=32, p=3)
    o, A = oracle.OracleH2(P, **prm), h2x.H2Matrix(P, **prm)
    B = W.rhs(2500, m, 601)
    for it in (1, 2, 3):
        X, info = h2x.block_cg_solve(A, torch.from_numpy(B).cuda(), rtol=1e-14, max_iter=it, variant="shared")
        ref, _ = o.block_cg_shared(B, rtol=1e-14, max_iter=it)
        err = np.linalg.norm(X.cpu().numpy() - ref, axis=0) / np.linalg.norm(ref, axis=0)
        print(f"m={m} it={it} err={err.max():.2e}")
        assert info.iters == it and err.max() <= 1e-12


@pytest.mark.parametrize("m", [9, 40, 64])
def test_dependent_columns(m):
    import paper_2509_17257_amd as h2x
    P = W.sphere_points(2000, 610)
    prm = dict(ell=0.5, shift=1.0, eta=1.0, leaf=32, p=3)
    o, A = oracle.OracleH2(P, **prm), h2x.H2Matrix(P, **prm)
    B = W.rhs(2000, m, 611)
    B[:, m - 1] = 2.0 * B[:, 0] - B[:, 1]  # dependent
    B[:, m // 2] = 0.0
    B[:, 3] = B[:, 2]
    X, info = h2x.block_cg_solve(A, torch.from_numpy(B).cuda(), rtol=1e-8, variant="shared")
    R = B - o.matmul(X.cpu().numpy())
    nb = np.linalg.norm(B, axis=0)
    nb[nb == 0] = 1.0
    assert info.status == 0 and (np.linalg.norm(R, axis=0) / nb).max() <= 2e-8
