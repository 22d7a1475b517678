"""Translations by rotation (k_fmm_m2l.hip) where most boxes hold no points: sheets and chains of
bodies, so that most displacements of a workgroup lead to empty boxes and most of its own four
boxes may be empty.  Eight waves (orders to 12) and four (above), levels 2 to 5.
Against the oracle's FMM to level 3; above, where that takes minutes (it translates every box),
against the float64 sum on the same tree, whose translations are the dense ones.

Tolerance: float32 rounding, 2e-5 of the largest value as for the same comparison on full cubes.

The time: the float64 sum takes the dense translations, which leave out the boxes without
points and need more operations at every pair of boxes; the float32 sum of the same points, with the
same tree, cannot take longer unless it works on empty boxes (it took 1.5 times as long then)."""
import math
import time

import numpy as np
import pytest

from oracle import fmm
from tests.test_gpu_fmm import _ctx, _dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _bodies(kind, n, npts, seed):
    """n unit spheres of npts Fibonacci points, 2.75 apart: in a plane, along x, along the diagonal."""
    rng = np.random.default_rng(seed)
    k = np.arange(npts) + 0.5
    th, ph = np.arccos(1 - 2 * k / npts), math.pi * (1 + 5 ** 0.5) * k
    u = np.stack([np.sin(th) * np.cos(ph), np.sin(th) * np.sin(ph), np.cos(th)], 1)
    i, side = np.arange(n), math.ceil(n ** 0.5)
    c = {"sheet": [i % side, i // side, 0 * i], "chain": [i, 0 * i, 0 * i], "diagonal": [i, i, i]}[kind]
    X = (2.75 * np.stack(c, 1)[:, None, :] + u).reshape(-1, 3)
    return X, np.tile(u, (n, 1)), rng.standard_normal(X.shape), np.repeat(i, npts)


@pytest.mark.parametrize("kind,n,P,max_level", [("sheet", 100, 5, 3), ("sheet", 49, 12, 3), ("chain", 20, 8, 3),
                                                ("chain", 20, 13, 3), ("diagonal", 9, 14, 2)])
def test_empty_boxes(kind, n, P, max_level):
    print(f"\n[case] fmm on a {kind} of {n}, order {P}, max_level={max_level}", flush=True)
    X, Nn, q, body = _bodies(kind, n, 16, 7 + P)
    ref, (_, _, L) = fmm.traction(X, Nn, q, body, P, 2.0, L_max=max_level)
    s = _ctx((X.shape[0] // 40 // 4 + 1) * 4, 4, P, max_level)
    y, lev = s.far_traction_fmm(_dev(X), _dev(Nn), _dev(q), 16, 2.0, precision=1)
    s.close()
    assert lev == L == max_level
    assert np.abs(y.cpu().numpy().T - ref).max() < 2e-5 * np.abs(ref).max()


@pytest.mark.parametrize("kind,n,P", [("sheet", 900, 12), ("sheet", 1600, 15), ("chain", 64, 12), ("chain", 40, 13),
                                      ("diagonal", 40, 12), ("diagonal", 100, 9)])
def test_empty_boxes_of_deep_trees(kind, n, P):
    print(f"\n[case] fmm on a {kind} of {n}, order {P}, float32 against float64", flush=True)
    X, Nn, q, _ = _bodies(kind, n, 16, 7 + P)
    s = _ctx((X.shape[0] // 40 // 4 + 1) * 4, 4, P)
    Xd, Nd, qd = _dev(X), _dev(Nn), _dev(q)
    (ref, lev), (y, lev32) = (s.far_traction_fmm(Xd, Nd, qd, 16, 2.0, precision=k) for k in (0, 1))
    s.close()
    assert lev == lev32 >= 4
    assert float((y - ref).abs().max()) < 2e-5 * float(ref.abs().max())


def test_time_on_a_diagonal():
    print("\n[case] fmm on a diagonal of 100, order 12: float32 against float64", flush=True)
    X, Nn, q, _ = _bodies("diagonal", 100, 60, 3)
    s = _ctx(20, 12, 12)
    Xd, Nd, qd = _dev(X), _dev(Nn), _dev(q)
    best = []
    for prec in (0, 1):
        t = []
        for _ in range(10):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            _, lev = s.far_traction_fmm(Xd, Nd, qd, 60, 2.0, precision=prec)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        assert lev >= 5
        best.append(min(t))
    s.close()
    assert best[1] < best[0]
