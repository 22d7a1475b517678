"""Block inverses (k_inverse.hip) at the sizes where its panels, sub-panels and strips change:
3M = 36 (less than a panel), 72, 216 (a panel of 24 at the end), 936, 1020 and above 1024 and 2048
rows (two and three rows per thread), for one shape and for several, against the inverse of
the context's own A0 by LAPACK.

Tolerance: A0 is a second-kind operator of condition number below 100 here; two inverses by
partial pivoting differ by about n eps cond: 3000 x 2.2e-16 x 100 = 7e-11 in the worst case; 1e-11
of the largest entry."""
import numpy as np
import pytest

from paper_1606_07428_amd import inputs, rbm

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("p,n", [(2, 1), (3, 2), (5, 3), (8, 2), (12, 1), (13, 2), (16, 2), (18, 1), (20, 1)])
def test_block_inverse(p, n):
    print(f"\n[case] block inverse p={p} shapes={n}", flush=True)
    w = inputs.tiny(n=n, p=p, seed=40 + p, lmax=min(3, p - 2))
    s = rbm.solver_for(w, max_iter=2, p_sing=0 if p <= 13 else p + 1)
    M3 = 3 * s.M
    A = s.read("A0", n * M3 * M3).reshape(n, M3, M3)
    P = s.read("P0", n * M3 * M3).reshape(n, M3, M3)
    s.close()
    for a, q in zip(A, P):
        ref = np.linalg.inv(a)
        assert np.linalg.cond(a, 1) < 1e4
        assert np.abs(q - ref).max() < 1e-11 * np.abs(ref).max()
