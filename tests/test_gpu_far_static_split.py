"""The ordered sum of the no-allocation entry point: bitwise the context's in float32 at the sizes whose
96 slots take more than 64 MiB (28,436 to 28,671 points), and at a float64 size whose unordered pairs do not fit
its scratch, against the oracle's direct sum at sampled targets (1e-12 of the largest output: the
square root of 7 x 10^5 terms times 2^-53 is 9e-14)."""
import numpy as np
import pytest

from paper_1606_07428_amd import rbm
from oracle import farfield as ff
from tests.helpers import rel_err
from tests.test_gpu_far_sizes import _context, _dev, _points

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [28436, 28500, 28671])
def test_float32_equals_the_context(n):
    print(f"\n[case] static against context, float32, n={n}", flush=True)
    _, X, Nn, q = _points(n, n)
    a = (_dev(X.T), _dev(Nn.T), _dev(q.T))
    s = _context(n)
    y = s.far_traction(*a, 312, precision=1)
    ys = rbm.far_traction_static(*a, 312, precision=1)
    assert torch.equal(y, ys)
    s.close()


def test_ordered_sum_of_the_largest_inputs():
    n, M = 720000, 312
    print(f"\n[case] static sum n={n} float64, ordered", flush=True)
    rng, X, Nn, q = _points(n, n)
    y = rbm.far_traction_static(_dev(X.T), _dev(Nn.T), _dev(q.T), M).cpu().numpy().T
    idx = np.unique(np.concatenate([rng.choice(n, 24, replace=False), [0, n - 1]]))
    body = np.arange(n) // M
    assert rel_err(y[idx], ff.traction_sum(X[idx], Nn[idx], X, q, body[idx], body)) < 1e-12
