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


# every class of split takes the register passes; 512, 640, 720 and lengths above 729 have none
@pytest.mark.parametrize("M,grid,same", [
    ((45, 45), None, False), ((81, 1125), None, False), ((1125, 243), None, False), ((225, 135), None, False),
    ((405, 375), None, False), ((729, 625), None, False), ((1125, 1125), None, True),
    ((1125, 1125), (512, 512), True), ((1875, 1875), (640, 640), True), ((1875, 1875), (720, 720), True),
    ((1215, 1215), (600, 500), False), ((1215, 1215), (576, 480), False)])
def test_lengths_with_a_split(M, grid, same, monkeypatch):
    N = tuple(g - 1 for g in grid) if grid else tuple((m + 1) // 4 * 2 - 1 for m in M)
    pb = _problem(N, M, False)
    if grid:
        cell = homgen.square_inclusion_cell(2, side=0.5, rho_in=12.0, Y=np.array(pb.Y))
        pb.set_gani_from_cell(cell, grid=grid)
    for dual in (False, True):
        x = _fields(pb, dual)[0]
        a, b = _both(monkeypatch, lambda: pb.apply(x, dual).cpu().numpy())
        _check(a, b, same)


# mixed mode: a specialised pass on one 2D axis and register passes on the other share a pack-major buffer.
# FP32 operator 2e-6 and bounds of whole solves 1e-6, as for two specialised passes
@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("N,M", [((13, 23), (25, 45)), ((41, 121), (81, 243)), ((63, 113), (125, 225)),
                                 ((23, 13), (45, 25)), ((121, 41), (243, 81)), ((113, 63), (225, 125))])
def test_mixed_routes(N, M, full, monkeypatch):
    import paper_1404_3614_amd as H
    cell = homgen.Inclusions(d=2, Y=np.array([1.0, 1.3]), A0=np.eye(2))
    cell.add("rect", [0.2, -0.1], [0.3, 0.5], np.diag([4.0, 9.0]) if full else 12.0 * np.eye(2))
    pb = H.problem_from_cell(cell, N, precision="mixed", M=M)
    for dual in (False, True):
        x = _fields(pb, dual)[0]
        a, b = _both(monkeypatch, lambda: pb.apply(x, dual).cpu().numpy())
        assert np.abs(a - b).max() <= 2e-6 * np.abs(b).max() and not np.array_equal(a, b)
    exact = H.problem_from_cell(cell, N, precision="fp64", M=M)
    monkeypatch.setenv("HOM_NO_FAST", "1")
    ref = exact.solve_bounds(tol=1e-8)
    monkeypatch.delenv("HOM_NO_FAST")
    got = pb.solve_bounds(tol=1e-8)
    for k in ("A_up", "A_low"):
        assert np.abs(got[k] - ref[k]).max() <= 1e-6 * np.abs(ref[k]).max()
