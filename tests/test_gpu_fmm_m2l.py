"""Translations by rotation (k_fmm_m2l.hip) at every order they take (2..15) and the dense ones beyond
(16), levels 2 to 4, against the oracle's FMM on the same tree and order, with boxes without points.

Tolerance: float32 rounding, 2e-5 of the largest value as for the same comparison elsewhere; the
rotations are orthogonal, so their rounding is no larger than the dense sums'."""
import numpy as np
import pytest

from oracle import fmm
from tests.test_gpu_fmm import _cloud, _ctx, _dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("P,side,max_level", [(P, 6, 3) for P in range(2, 17)] + [(6, 4, 2), (12, 4, 2), (9, 12, 4)])
def test_translations(P, side, max_level):
    print(f"\n[case] fmm translations: order {P} side={side} max_level={max_level}", flush=True)
    X, Nn, q, body = _cloud(side, 3.4, 12, 100 + P)
    keep = np.ones(side ** 3, bool)
    keep[::3] = False                       # gaps in the cloud: boxes without points
    sel = keep[body]
    X, Nn, q = X[sel], Nn[sel], q[sel]
    body = np.repeat(np.arange(int(keep.sum())), 12)
    ref, (_, _, L) = fmm.traction(X, Nn, q, body, P, 2.0, L_max=max_level)
    s = _ctx((X.shape[0] // 40 // 4 + 1) * 4, 4, P, max_level)
    y, lev = s.far_traction_fmm(_dev(X), _dev(Nn), _dev(q), 12, 2.0, precision=1)
    s.close()
    assert lev == L == max_level
    assert np.abs(y.cpu().numpy().T - ref).max() < 2e-5 * np.abs(ref).max()
