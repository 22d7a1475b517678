"""The traction sum of the no-allocation entry point where its scratch holds only part of the block rows
at a time (several phases; chunks and grids of their own), against the oracle's direct sums at
sampled targets, and its time against the context's sum of the same points, which runs in one phase.

Tolerances as for the sums of one phase: float64 1e-12 of the largest output (the square root of 3 x 10^5
terms times 2^-53 is 6e-14), float32 arithmetic on float32-rounded inputs 1e-5.
Time: the phases read and write every output once more and each ends on the drain of the chip, together
some 10 %; 1.2 times the context's (grids that left half of the shader engines idle in a
phase's first and last blocks took 1.32 and 1.45)."""
import time

import numpy as np
import pytest

from paper_1606_07428_amd import rbm
from oracle import farfield as ff
from tests.helpers import rel_err
from tests.test_gpu_far_sizes import _context, _dev, _points

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,M,prec", [(69001, 312, 1), (75003, 5000, 1), (112606, 312, 1), (73000, 1, 0), (96010, 312, 0),
                                      (171274, 312, 1), (300007, 312, 0)])
def test_phases(n, M, prec):
    print(f"\n[case] static sum in phases n={n} M={M} precision={prec}", flush=True)
    rng, X, Nn, q = _points(n, n + M)
    add = rng.standard_normal((n, 3))
    a = (_dev(X.T), _dev(Nn.T), _dev(q.T))
    y = rbm.far_traction_static(*a, M, add=_dev(add.T), precision=prec).cpu().numpy().T
    if prec:
        X, Nn, q = (v.astype(np.float32).astype(np.float64) for v in (X, Nn, q))
    idx = np.unique(np.concatenate([rng.choice(n, 48, replace=False), [0, n - 1, n // 2]]))
    body = np.arange(n) // M
    ref = ff.traction_sum(X[idx], Nn[idx], X, q, body[idx], body)
    assert rel_err(y[idx] - add[idx], ref) < (1e-12 if prec == 0 else 1e-5)


@pytest.mark.parametrize("n,prec", [(96010, 0), (171274, 1)])
def test_time_of_phases(n, prec):
    print(f"\n[case] time of the static sum in phases n={n} precision={prec}", flush=True)
    _, X, Nn, q = _points(n, n)
    a = (_dev(X.T), _dev(Nn.T), _dev(q.T))
    s = _context(n)
    best = []
    for f in (lambda: s.far_traction(*a, 312, precision=prec), lambda: rbm.far_traction_static(*a, 312, precision=prec)):
        t = []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            f()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        best.append(min(t))
    s.close()
    assert best[1] < 1.2 * best[0]
