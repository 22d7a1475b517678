"""Leaf evaluation of the fast multipole far field with 16, 8 and 4 waves per work item (512, 4094
and 4182 work items of 64 targets), against the oracle's FMM on the same tree and order.  Leaves
hold parts of several bodies, so groups of sources with and without points of the targets'
bodies occur, whole and partial ones.

Tolerance: rounding, as for the same comparison on smaller trees (float64 sums of 1e4 terms with
cancellation 1e-12, float32 2e-5 of the largest value)."""
import numpy as np
import pytest

from oracle import fmm
from tests.test_gpu_fmm import _cloud, _ctx, _dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("side,npts,max_level", [(6, 33, 3), (12, 16, 4), (12, 80, 4)])
def test_leaf_sums(side, npts, max_level):
    print(f"\n[case] fmm leaves: side={side} npts={npts} max_level={max_level}", flush=True)
    X, Nn, q, body = _cloud(side, 3.0, npts, 5 + side)
    ref, (_, _, L) = fmm.traction(X, Nn, q, body, 4, 2.0, L_max=max_level)
    s = _ctx((X.shape[0] // 84 // 4 + 1) * 4, 6, 4, max_level)
    for prec, tol in ((0, 1e-12), (1, 2e-5)):
        y, lev = s.far_traction_fmm(_dev(X), _dev(Nn), _dev(q), npts, 2.0, precision=prec)
        assert lev == L == max_level
        assert np.abs(y.cpu().numpy().T - ref).max() < tol * np.abs(ref).max()
    s.close()
