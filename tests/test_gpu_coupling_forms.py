"""Launch shapes of the FP64 coupling stage: every one gives the same bits.

The list of a row cluster is summed in four consecutive parts added in order, whatever number
of column tiles, waves or work-groups the launch takes, so a product of the first columns of X
equals the first columns of the product, a forced tile width equals the built-in rule, and a
system in a merged plan equals the system alone -- bit for bit, at sizes on both sides of the
rules (few rows: tiles and narrow slabs; many rows: wide slabs and a narrow last slab).
"""
import numpy as np
import pytest

import oracle
from paper_2509_17257_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _h2x():
    import paper_2509_17257_amd as h2x
    return h2x


# orders, leaves and sizes below and above the thresholds of each rule
SIZES = [(1, 8, 700), (2, 16, 900), (2, 16, 9000), (3, 32, 1200), (3, 32, 14000), (4, 64, 1500), (4, 64, 26000),
         (5, 64, 1500), (5, 64, 9000)]


@pytest.mark.parametrize("p,leaf,n", SIZES, ids=[f"p{s[0]}-n{s[2]}" for s in SIZES])
def test_shapes_agree(p, leaf, n):
    h2x = _h2x()
    P = W.sphere_points(n, 500 + p)
    prm = dict(ell=0.5, shift=1.0, eta=1.0, leaf=leaf, p=p)
    A = h2x.H2Matrix(P, **prm)
    assert A.plan.n_adm > 0
    X = torch.from_numpy(W.rhs(n, 100, 501)).cuda()
    Y = h2x.h2_matmul(A, X)
    if n < 5000:
        ref = oracle.OracleH2(P, **prm).matmul(X.cpu().numpy())
        err = np.linalg.norm(Y.cpu().numpy() - ref, axis=0) / np.linalg.norm(ref, axis=0)
        assert err.max() <= 1e-12
    for m in (1, 16, 17, 33, 50, 64, 65, 81):
        Xm = X[:, :m].contiguous()
        Ym = h2x.h2_matmul(A, Xm)
        # the other stages' sums do not depend on the column count either
        assert torch.equal(Ym, Y[:, :m]), m
        for nj in range(1, min(4, (m + 15) // 16) + 1):
            A.set_tune(m, nj_coupling=nj)
            assert torch.equal(h2x.h2_matmul(A, Xm), Ym), (m, nj)
        A.set_tune(m)


@pytest.mark.parametrize("p,leaf", [(2, 16), (3, 32), (4, 64), (5, 64)])
def test_merged_equals_single(p, leaf):
    h2x = _h2x()
    sizes = (600, 4000, 1500, 12000)
    pts = [W.sphere_points(n, 510 + i) for i, n in enumerate(sizes)]
    prms = [dict(ell=0.3 + 0.1 * i, shift=1.0, eta=1.0, leaf=leaf, p=p) for i in range(len(sizes))]
    plans = [h2x.Plan(q, **prm) for q, prm in zip(pts, prms)]
    merged = h2x.H2Matrix(h2x.Plan.merge(plans))
    X = torch.from_numpy(W.rhs(sum(sizes), 20, 520)).cuda()
    Y = h2x.h2_matmul(merged, X)
    a = 0
    for q, prm in zip(pts, prms):
        A = h2x.H2Matrix(q, **prm)
        assert torch.equal(h2x.h2_matmul(A, X[a:a + len(q)].contiguous()), Y[a:a + len(q)])
        a += len(q)
