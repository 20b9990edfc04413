"""GPU: which FP64 passes the register transforms take.  The lengths of the other
axes have no split (1125) or no register row pass, so that a whole call runs the
generic passes exactly if the pass in question does: its results are then those
of HOM_NO_FAST (read at each call) to the bit, and differ in the last bits
otherwise.  The register route's values stay within 1e-12 of the generic ones
(two routes of the same FP64 arithmetic)."""
import numpy as np
import pytest

import homgen

pytestmark = pytest.mark.gpu


def _problem(N, M, full, seed=3):
    import paper_1404_3614_amd as H
    if len(N) == 3:
        cell = homgen.sphere_cell(seed=seed, n=5, anisotropic=full)
    else:
        cell = homgen.Inclusions(d=2, Y=np.array([1.0, 1.3]), A0=np.eye(2))
        cell.add("rect", [0.2, -0.1], [0.3, 0.5], np.diag([4.0, 9.0]) if full else 12.0 * np.eye(2))
    return H.problem_from_cell(cell, N, precision="fp64", M=M)


def _both(monkeypatch, call):
    out = []
    for generic in (False, True):
        if generic:
            monkeypatch.setenv("HOM_NO_FAST", "1")
        else:
            monkeypatch.delenv("HOM_NO_FAST", raising=False)
        out.append(call())
    return out


def _fields(pb, dual):
    import torch
    rng = np.random.default_rng(5)
    n = pb.flen[int(dual)]
    return [torch.tensor(rng.standard_normal(n) + 1j * rng.standard_normal(n), device="cuda") for _ in range(pb.d)]


def _check(a, b, same):
    assert np.isfinite(a).all() and np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
    assert np.array_equal(a, b) == same


# 25 * 5 on a 3D axis: rows of more than 256 pairs, and columns beyond one round of blocks, stay generic
@pytest.mark.parametrize("dual", [False, True])
@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("N,M,same", [
    ((23, 23, 3), (125, 1125, 125), True), ((3, 3, 3), (125, 1125, 125), False),
    ((23, 23, 3), (81, 1125, 125), False), ((23, 23, 3), (125, 1125, 135), False)])
def test_operator_route(N, M, same, full, dual, monkeypatch):
    pb = _problem(N, M, full)
    x = _fields(pb, dual)[0]
    a, b = _both(monkeypatch, lambda: pb.apply(x, dual).cpu().numpy())
    _check(a, b, same)


# the quadrature of the bounds: registers in 2D but for 25 * 5 (generic rows with it), in 3D where a block of the
# register pass has a grid point per thread
@pytest.mark.parametrize("dual", [False, True])
@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("N,M,same", [
    ((23, 13), (625, 1125), False), ((187, 13), (375, 1125), False), ((13, 13), (25, 1125), False),
    ((63, 13), (125, 1125), True), ((63, 41), (125, 81), True), ((41, 63), (81, 125), False),
    ((5, 187, 3), (9, 1125, 125), True), ((23, 23, 3), (75, 1125, 125), True), ((23, 23, 3), (81, 1125, 125), False)])
def test_quadrature_route(N, M, same, full, dual, monkeypatch):
    pb = _problem(N, M, full)
    x = _fields(pb, dual)
    a, b = _both(monkeypatch, lambda: pb.bounds(None, x)["B_up"] if dual else pb.bounds(x, None)["A_up"])
    _check(a, b, same)
