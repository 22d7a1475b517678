"""GMRES on vectors short enough for the one-workgroup Arnoldi step, on both sides of its limits
(length 5120, length times vectors 81920: 4752 crosses the latter within a cycle), against the
oracle's dense solution.

Tolerance: the solution is converged to 1e-13 of the right-hand side and the operators agree to
1e-12 with the oracle's; condition numbers below 100: 1e-10, as for the same comparison elsewhere."""
import pytest

from oracle import system as sy
from paper_1606_07428_amd import inputs, rbm
from tests.helpers import oracle_problem, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,p,max_iter", [(2, 2, 100), (3, 5, 7), (9, 8, 100), (11, 8, 100), (12, 8, 100)])
def test_short_vectors(n, p, max_iter):
    print(f"\n[case] short Krylov vectors n={n} p={p} max_iter={max_iter}", flush=True)
    w = inputs.tiny(n, p, seed=70 + n, lmax=min(3, p - 2))
    s = rbm.solver_for(w, tol=1e-13, max_iter=max_iter, max_restart=60)
    VW, info = s.solve(w["FT"])
    s.close()
    print(f"[case] iterations {info['iters']} cycles {info['cycles']}", flush=True)
    assert info["rel_residual"] < 1e-13
    assert rel_err(VW, sy.solve_dense(oracle_problem(w), w["FT"])[2]) < 1e-10
