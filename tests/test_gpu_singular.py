"""Singular self operators (k_singular.hip) at the sizes where its tiles change: 32 x 32 tiles of
the rotated grid (p_sing + 1 = 32, 33, 34 and the largest), 16-wide tiles of m (p + 1 = 16, 17)
and the passes over (l, m) (p = 12, 13, 15, 16, 20), against the oracle: rows of A0 for targets at
both ends and the middle of the grid, and for the smaller sizes the velocity functional, which
sums every row of the single layer.

Tolerance: sums of at most 2 x 64 x 65 rounded terms (sqrt(8320) eps = 2e-14), four contractions
one after the other and a kernel that loses up to a digit near the pole (r from x_t - x):
1e-12 of the largest entry."""
import numpy as np
import pytest

from helpers import oracle_shapes, rel_err
from oracle import singular as sg
from paper_1606_07428_amd import inputs, rbm

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _functional(shape):
    g = shape.geom
    M = g["w"].size
    G = np.zeros((6, 3 * M))
    for c in range(3):
        G[c, c * M:(c + 1) * M] = g["w"] / g["area"]
        e = np.zeros(3)
        e[c] = 1.0
        G[3:, c * M:(c + 1) * M] = np.linalg.inv(g["tau"]) @ (g["w"] * np.cross(g["r"], e[:, None], axis=0))
    return G @ shape.ops["S"]


@pytest.mark.parametrize("p,ps", [(2, 3), (3, 6), (4, 31), (5, 32), (6, 33), (8, 64), (12, 24), (13, 14), (15, 17),
                                  (16, 17), (16, 32), (20, 21), (20, 40)])
def test_singular_operators(p, ps):
    print(f"\n[case] singular operators p={p} p_sing={ps}", flush=True)
    w = inputs.tiny(n=2, p=p, seed=60 + p, lmax=min(3, p - 2))
    s = rbm.solver_for(w, max_iter=2, p_sing=ps)
    M, M3 = s.M, 3 * s.M
    A = s.read("A0", 2 * M3 * M3).reshape(2, M3, M3).transpose(0, 2, 1)
    V = s.read("V0", 2 * 6 * M3).reshape(2, 6, M3)
    s.close()
    whole = p <= 8 or (p, ps) in ((13, 14), (16, 17))
    for k, sh in enumerate(oracle_shapes(w, with_ops=False, ps=ps)):
        if whole:
            sh.ops = sg.singular_operators(sh.coef, p, ps, w.get("eta", 1.0))
            assert rel_err(V[k], _functional(sh)) < 1e-12
        L = sg.L_operator(sh.geom)
        targets = [0, 1, 2 * p, M // 2 + 1, M - 2 * p - 1, M - 1]
        rows = sg.singular_rows(sh.coef, p, ps, targets, which=("K",))["K"]
        for i, t in enumerate(targets):
            at = [c * M + t for c in range(3)]
            ref = rows[i].reshape(3, M3) + L[at]
            ref[np.arange(3), at] += 0.5
            assert rel_err(A[k][at], ref) < 1e-12
