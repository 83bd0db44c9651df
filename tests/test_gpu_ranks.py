"""GPU parity of the ranks above 64 (Chebyshev orders 5 to 8) against the CPU oracle.

Per column and per entry <= 1e-12 (the bound of the other FP64 products) at ranks whose last
16-row tile, 8-column pair or 64-column chunk is partial (125, 216, 343) or full (512), column
counts around the tile widths, leaves of several 64-row chunks, alpha / beta and tree order;
the coupling matrices read and written back through the padded layout.
"""
import numpy as np
import pytest

import oracle
from paper_2509_17257_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12


def _h2x():
    import paper_2509_17257_amd as h2x
    return h2x


def _err(a, b):
    d = np.abs(a - b).max(axis=0) / np.maximum(np.abs(b).max(axis=0), 1e-300)
    c = np.linalg.norm(a - b, axis=0) / np.maximum(np.linalg.norm(b, axis=0), 1e-300)
    return max(d.max(), c.max())


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


CASES = [(5, 64, 2500, 1), (5, 128, 3000, 16), (5, 64, 2500, 17), (5, 128, 4000, 64), (5, 150, 3000, 70),
         (6, 64, 1500, 3), (6, 128, 2000, 33), (7, 128, 1500, 5), (8, 128, 1200, 18)]


@pytest.mark.parametrize("p,leaf,n,m", CASES, ids=[f"p{c[0]}-leaf{c[1]}-m{c[3]}" for c in CASES])
def test_products_match_oracle(p, leaf, n, m):
    h2x = _h2x()
    P = W.line_points(n, 300 + p) + 0.05 * W.cube_points(n, 301 + p)  # long: admissible blocks on many levels
    prm = dict(ell=0.5, shift=1.0, eta=1.0, leaf=leaf, p=p)
    o, A = oracle.OracleH2(P, **prm), h2x.H2Matrix(P, **prm)
    assert o.n_adm > 0
    X, Y0 = W.rhs(n, m, 302), W.rhs(n, m, 303)
    ref = o.matmul(X)
    errs = [_err(h2x.h2_matmul(A, _dev(X)).cpu().numpy(), ref)]
    out = _dev(Y0)
    h2x.h2_matmul(A, _dev(X), alpha=-1.5, beta=0.5, out=out)
    errs.append(_err(out.cpu().numpy(), 0.5 * Y0 - 1.5 * ref))
    q = A.plan.perm()
    errs.append(_err(h2x.h2_matmul(A, _dev(X[q]), tree_order=True).cpu().numpy(), ref[q]))
    print(f"p={p} leaf={leaf} m={m} adm={o.n_adm}: {errs}")
    assert max(errs) <= TOL
    # coupling matrices through the padded layout: read, scaled, written back
    S = A.coupling()
    A.set_coupling(2.0 * S)
    assert torch.equal(A.coupling(), 2.0 * S)
    A.set_coupling(S)
    assert _err(h2x.h2_matmul(A, _dev(X)).cpu().numpy(), ref) <= TOL
