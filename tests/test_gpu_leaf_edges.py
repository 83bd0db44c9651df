"""Leaf stage, column halves for three row tiles: a last slab of at most half the slab's columns (the
second half would start past X's row) and one of just more than half.

FP64: slabs of 32 columns forced at 33 to 49 columns, the same bits as the built-in slabs (the
sums do not depend on the slab).  FP32 and BF16: 145 to 177 columns are slabs of 64; against
leaf_kind 1, which differs by the order of the FP32 sums only (1e-5, as in the other tests)."""
import numpy as np
import pytest

from paper_2509_17257_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaf", [40, 45, 100])
def test_fp64_narrow_last_slab(leaf):
    import paper_2509_17257_amd as h2x
    n = 2300
    A = h2x.H2Matrix(W.cube_points(n, 750), ell=0.4, shift=1.0, eta=1.0, leaf=leaf, p=3)
    X = torch.from_numpy(W.rhs(n, 49, 751)).cuda()
    for m in (33, 47, 48, 49):
        Xm = X[:, :m].contiguous()
        Y = h2x.h2_matmul(A, Xm)
        A.set_tune(m, np_leaf=1)
        assert torch.equal(h2x.h2_matmul(A, Xm), Y), m
        A.set_tune(m)


@pytest.mark.parametrize("leaf", [16, 40, 45, 100])
@pytest.mark.parametrize("prec", ["f32", "bf16"])
def test_lowp_narrow_last_slab(leaf, prec):
    import paper_2509_17257_amd as h2x
    n = 2300
    A = h2x.H2Matrix(W.cube_points(n, 752), storage=prec, ell=0.4, shift=1.0, eta=1.0, leaf=leaf, p=3)
    X = torch.from_numpy(W.rhs(n, 177, 753)).cuda()
    for m in (145, 160, 161, 177):
        Xm = X[:, :m].contiguous()
        A.set_tune(m, leaf_kind=1)
        ref = h2x.h2_matmul(A, Xm)
        A.set_tune(m)
        Y = h2x.h2_matmul(A, Xm)
        assert (torch.linalg.norm(Y - ref, dim=0) / torch.linalg.norm(ref, dim=0)).max().item() <= 1e-5, m
