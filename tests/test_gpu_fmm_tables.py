"""The rotation tables of the float32 translations are made for float32 sums alone: the bytes of
the workspace that a call writes.  343 displacements x 2 tables x 40 groups of 64 lanes x 4 floats are
28 MB; all else that a call of this size writes (dense tables of two levels, expansions,
sorted points) is below 16 MB."""
import pytest

from tests.test_gpu_fmm import _cloud, _ctx, _dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_float64_sums_make_no_float32_tables():
    print("\n[case] workspace bytes written by a float64 and a float32 fmm sum, order 12, 3 levels", flush=True)
    X, Nn, q, _ = _cloud(6, 3.4, 12, 5)
    s = _ctx(68, 4, 12, 3)
    written, out = [], []
    for prec in (0, 1):
        torch.cuda.synchronize()
        s.ws.fill_(0xA5)
        y, lev = s.far_traction_fmm(_dev(X), _dev(Nn), _dev(q), 12, 2.0, precision=prec)
        assert lev == 3
        written.append(int((s.ws != 0xA5).sum()))
        out.append(y)
    s.close()
    assert written[0] < 20e6 < written[1]
    assert float((out[0] - out[1]).abs().max()) < 2e-5 * float(out[0].abs().max())
