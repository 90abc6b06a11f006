"""TV solves on the formed normal matrix at the edges of its tiles: one block of 64 and its
neighbours, block rows that fill and leave groups of the factor, columns that leave a ragged tile of
64 and of 128, and matrices large enough for tiles of 128 in the normal matrix (3,969 unknowns)
and in the factor's updates (4,289)."""
import numpy as np
import pytest

from oracle import tv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mgrt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_04605_amd as m
    return m


@pytest.mark.parametrize("M,rows,prec", [
    (1, 7, 64), (17, 20, 32), (63, 64, 32), (64, 95, 64), (65, 97, 32), (127, 128, 64), (128, 4000, 32),
    (129, 161, 32), (191, 400, 64), (192, 193, 32), (193, 5000, 64), (1000, 2111, 32), (1537, 1601, 64),
    (3101, 3333, 32)])
def test_direct_solve(mgrt, M, rows, prec):
    """One step against the oracle's dense solve.  A Gaussian L of these shapes leaves the matrix a
    condition number up to about 1e5: 1e5 * 2^-53 times a modest power of M, <= 1e-9."""
    rng = np.random.default_rng(M + rows)
    L = rng.normal(size=(rows, M))
    if prec == 32:
        L = L.astype(np.float32)
    r = rng.normal(size=rows)
    rp, col, val = np.arange(M + 1), np.arange(M), np.ones(M)
    ref = tv.tv_iterates(L.astype(np.float64), r, np.eye(M), 0.5, 1)[0]
    z, its = mgrt.Context(0).tv_invert_level(L, r, rp, col, val, 0.5, iters=1)
    assert its[0] == 0
    err = float(np.linalg.norm(z[0] - ref) / np.linalg.norm(ref))
    print(f"M={M} rows={rows} fp{prec}: {err:.2e}")
    assert err <= 1e-9


@pytest.mark.parametrize("M,rows,prec", [(3969, 5200, 32), (4289, 5600, 64), (4300, 5600, 32), (4353, 5700, 64)])
def test_direct_solve_in_tiles_of_128(mgrt, M, rows, prec):
    """One step where whole tiles of 128 and the quarters behind them meet a ragged edge, in the
    normal matrix (all) and in the factor (from 4,289).  A Gaussian L with 1.3 M rows leaves the
    matrix a condition number of about 250: 250 * 2^-53 * M <= 2e-10."""
    rng = np.random.default_rng(M)
    L = rng.normal(size=(rows, M))
    if prec == 32:
        L = L.astype(np.float32)
    r = rng.normal(size=rows)
    ref = tv.tv_iterates(L.astype(np.float64), r, np.eye(M), 0.5, 1)[0]
    z, its = mgrt.Context(0).tv_invert_level(L, r, np.arange(M + 1), np.arange(M), np.ones(M), 0.5, iters=1)
    assert its[0] == 0
    err = float(np.linalg.norm(z[0] - ref) / np.linalg.norm(ref))
    print(f"M={M} rows={rows} fp{prec}: {err:.2e}")
    assert err <= 2e-10
