"""GPU: Fourier coefficients of matrix-inclusion cells whose table goes with the
launch (up to 24 inclusions for A and A^-1 together, 32 for one of them) or
through scratch (more), against the oracle, on rows shorter and longer than a
block.  A box term's error is the phase's, 2 pi 2u sum|n_a|, times its decay
prod min(h_a, 1/(pi n_a)): at most 8 u d per unit of |A_j| on either side, and
a few u for the factors and the sum: 1e-14 sum |A_j|."""
import numpy as np
import pytest

import homgen
from oracle import coefficients as co

pytestmark = pytest.mark.gpu


def _cell(d, n, iso, balls, seed):
    rng = np.random.default_rng(seed)
    spd = (lambda: float(rng.uniform(0.5, 4.0)) * np.eye(d)) if iso else (lambda: homgen.random_spd(rng, d, 0.5, 4.0))
    Y = np.array([1.0, 0.8, 1.2])[:d]
    c = homgen.Inclusions(d=d, Y=Y, A0=spd())
    for j in range(n):
        ball = balls and j % 3 != 0
        c.kind.append("ball" if ball else "rect")
        c.center.append(rng.uniform(-0.5, 0.5, d) * Y)
        c.size.append([float(rng.uniform(0.05, 0.3))] if ball else list(rng.uniform(0.05, 0.4, d)))
        c.A.append(spd())
    return c


@pytest.mark.parametrize("d,N,iso,balls,n", [
    (2, (13, 13), True, False, 0), (2, (13, 13), True, False, 1), (2, (23, 63), False, False, 24),
    (2, (5, 113), True, False, 25), (2, (13, 203), False, False, 32), (2, (63, 41), True, False, 33),
    (2, (5, 113), False, False, 70), (3, (5, 13, 5), True, True, 24), (3, (5, 5, 41), False, True, 25),
    (3, (13, 5, 13), False, True, 33), (3, (5, 5, 113), True, True, 3)])
def test_inclusion_coefficients(d, N, iso, balls, n):
    import paper_1404_3614_amd as H
    M = tuple(H.api.quad_grid(N))
    cell = _cell(d, n, iso, balls, seed=11 * n + d)
    Ah, Bh, nc = H.coef_from_cell(cell, N)
    assert nc == (1 if iso else d * (d + 1) // 2)
    comp = [(0, 0)] if nc == 1 else ([(0, 0), (1, 1), (0, 1)] if d == 2 else
                                     [(0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)])
    for inverse, pair in ((False, Ah), (True, Bh)):
        one = H.coef_inclusions(cell, N, nc, inverse)
        ref = co.fourier_coefficients(cell, M, inverse=inverse)
        f = np.linalg.inv if inverse else np.asarray
        tol = 1e-14 * (np.abs(f(cell.A0)).max() + sum(np.abs(f(A) - f(cell.A0)).max() for A in cell.A))
        for got in (pair, one):
            for c, (i, j) in enumerate(comp):
                assert np.abs(got[c].cpu().numpy() - ref[i, j]).max() <= tol, (inverse, c)


# above 600 blocks the blocks run across rows, from 5 points to longer than a block; below, whole rows per block
@pytest.mark.parametrize("N,M", [((3, 3), (405, 405)), ((3, 3), (729, 225)), ((3, 3, 3), (225, 225, 5)),
                                 ((3, 3, 3), (25, 81, 81)), ((3, 3, 3), (27, 45, 135)), ((3, 3), (375, 375)),
                                 ((3, 3, 3), (5, 9, 135)), ((3, 3), (5, 5))])
@pytest.mark.parametrize("iso,n", [(True, 5), (False, 40)])
def test_blocks_across_rows(N, M, iso, n):
    import paper_1404_3614_amd as H
    d = len(N)
    cell = _cell(d, n, iso, d == 3, seed=n + d)
    got = H.coef_from_cell(cell, N, M=M)
    comp = [(0, 0)] if iso else ([(0, 0), (1, 1), (0, 1)] if d == 2 else
                                 [(0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)])
    for inverse in (False, True):
        ref = co.fourier_coefficients(cell, M, inverse=inverse)
        f = np.linalg.inv if inverse else np.asarray
        tol = 1e-14 * (np.abs(f(cell.A0)).max() + sum(np.abs(f(A) - f(cell.A0)).max() for A in cell.A))
        for c, (i, j) in enumerate(comp):
            assert np.abs(got[int(inverse)][c].cpu().numpy() - ref[i, j]).max() <= tol, (inverse, c)
