"""All-pairs sums at the sizes where their split of the work changes: few points (chunks of
eight sources, one partial block), ragged last bodies and blocks, against the oracle's direct
sums at sampled targets.

Tolerances: a float64 sum of at most 10^5 terms carries at most about 10^5 x 2^-53 ~ 1e-11 of
the sum of magnitudes in the worst case and its square root in practice: 1e-12 of the largest
output.  Float32 arithmetic: the oracle gets the float32-rounded inputs, leaving 2^-24 per
operation and partial sums of at most 10^5 terms: 1e-5."""
import math

import numpy as np
import pytest

from paper_1606_07428_amd import rbm
from oracle import farfield as ff
from tests.helpers import rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")


def _context(n_points):
    p = 4
    M = 2 * p * (p + 1)
    w = {"p": p, "shapes": [("radial", [math.sqrt(4 * math.pi)])], "shape_id": np.zeros(1, np.int32),
         "centres": np.zeros((1, 3)), "quats": np.array([[1.0, 0, 0, 0]])}
    return rbm.solver_for(w, n_max=-(-n_points // M), max_iter=4)


def _points(n, seed):
    rng = np.random.default_rng(seed)
    side = max(1.0, (n / 4.0) ** (1 / 3))
    X = rng.uniform(0, side, (n, 3))
    Nn = rng.standard_normal((n, 3))
    Nn /= np.linalg.norm(Nn, axis=1)[:, None]
    return rng, X, Nn, rng.standard_normal((n, 3))


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,M", [(1, 1), (2, 1), (7, 3), (8, 1), (9, 4), (65, 16), (288, 144), (769, 60), (2051, 100),
                                 (5003, 312)])
def test_sums_at_small_and_ragged_sizes(n, M, prec):
    print(f"\n[case] far sums n={n} M={M} precision={prec}", flush=True)
    rng, X, Nn, q = _points(n, n + 7 * M + prec)
    s = _context(n)
    y = s.far_traction(_dev(X.T), _dev(Nn.T), _dev(q.T), M, precision=prec).cpu().numpy().T
    u = s.far_stokeslet(_dev(X.T), _dev(q.T), M, precision=prec).cpu().numpy().T
    ys = rbm.far_traction_static(_dev(X.T), _dev(Nn.T), _dev(q.T), M, precision=prec).cpu().numpy().T
    s.close()
    if prec:
        X, Nn, q = (a.astype(np.float32).astype(np.float64) for a in (X, Nn, q))
    assert np.array_equal(y, ys)
    idx = rng.choice(n, min(n, 64), replace=False)
    body = np.arange(n) // M
    rt = ff.traction_sum(X[idx], Nn[idx], X, q, body[idx], body)
    ru = ff.stokeslet_sum(X[idx], X, q, body[idx], body)
    if np.all(body == 0):
        assert not y.any() and not u.any()
        return
    tol = 1e-12 if prec == 0 else 1e-5
    assert rel_err(y[idx], rt) < tol and rel_err(u[idx], ru) < tol
