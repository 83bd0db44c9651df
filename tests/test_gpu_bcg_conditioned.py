"""Shared-space block CG where P^T A P is ill-conditioned without deflation (a small shift: condition
numbers of A of about 1e4 and 1e5): the solve converges to its tolerance on the true residual, in as
many iterations as the oracle's run of the method within 10 % (rounding alone moves the counts
by a few per cent)."""
import numpy as np
import pytest

import oracle
from paper_2509_17257_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [8, 33])
@pytest.mark.parametrize("ell,shift", [(0.5, 1e-1), (2.0, 1e-2)])
def test_small_shift(m, ell, shift):
    import paper_2509_17257_amd as h2x
    n = 2000
    P = W.sphere_points(n, 620)
    prm = dict(ell=ell, shift=shift, eta=1.0, leaf=32, p=3)
    o, A = oracle.OracleH2(P, **prm), h2x.H2Matrix(P, **prm)
    B = W.rhs(n, m, 621)
    X, info = h2x.block_cg_solve(A, torch.from_numpy(B).cuda(), rtol=1e-8, max_iter=600, variant="shared")
    _, ref = o.block_cg_shared(B, rtol=1e-8, max_iter=600)
    R = B - o.matmul(X.cpu().numpy())
    print(f"ell={ell} shift={shift} m={m}: {info.iters} iterations, oracle {ref['iters'] if isinstance(ref, dict) else ref.iters}")
    assert info.status == 0 and (np.linalg.norm(R, axis=0) / np.linalg.norm(B, axis=0)).max() <= 2e-8
    count = ref["iters"] if isinstance(ref, dict) else ref.iters
    assert abs(info.iters - count) <= max(2, 0.1 * count)
