"""The FP64 band product on the matrix cores (infoesrf_cov_apply) at the edges of its tiles:
64 rows a block, 16 rows and 16 systems a wavefront, the window in chunks of 16 positions, the
widths where it takes over from the plain kernel.  Against the dense P = L o (Z Z^T) in FP64; the
bound is that of two chains of rounded multiply-adds, (terms + N + 4) eps |P| |V| a component.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2503_00253_amd import infoesrf as ie  # noqa: E402

N = 7
CASES = [  # nz, nx, bz, bx, periodic z, periodic x
    (1, 63, 0, 8, 0, 1), (1, 65, 0, 31, 0, 0), (1, 129, 0, 32, 0, 1), (3, 50, 1, 9, 0, 1), (5, 37, 2, 18, 1, 1),
    (2, 257, 1, 40, 0, 0), (1, 400, 0, 159, 0, 1), (1, 161, 0, 80, 0, 1),
]


def problem(case):
    nz, nx, bz, bx, pz, px = case
    n = nz * nx
    rng = np.random.default_rng(n + bx)
    X = rng.standard_normal((n, N))
    table = rng.random((2 * bz + 1, 2 * bx + 1))
    table = table + table[::-1, ::-1]
    P = ie.Problem(torch.from_numpy(X).cuda(), np.arange(n + 1), np.arange(n), np.ones(n), np.full(n, 0.25), nz=nz,
                   nx=nx, periodic_z=pz, periodic_x=px, bz=bz, bx=bx, table=table)
    Z = (X - X.mean(axis=1, keepdims=True)) / np.sqrt(N - 1)
    L = np.zeros((n, n))
    for dz in range(-bz, bz + 1):
        for dx in range(-bx, bx + 1):
            for z in range(nz):
                zz = (z + dz) % nz if pz else z + dz
                if not 0 <= zz < nz:
                    continue
                x = np.arange(nx)
                xx = (x + dx) % nx if px else x + dx
                ok = (xx >= 0) & (xx < nx)
                L[z * nx + x[ok], zz * nx + xx[ok]] += table[dz + bz, dx + bx]
    return P, L * (Z @ Z.T), L


@pytest.mark.parametrize("B", [1, 16, 17, 65])
@pytest.mark.parametrize("case", CASES)
def test_band_product_matches_dense(case, B):
    print("[case] band product", case, B, file=sys.stderr, flush=True)
    P, dense, _ = problem(case)
    V = np.random.default_rng(B).standard_normal((P.n, B))
    V[:, B // 2] *= 1e-300
    got = ie.cov_apply(P, torch.from_numpy(V).cuda(), ie.default_opts()).cpu().numpy()
    terms = (2 * case[2] + 1) * (2 * case[3] + 1)
    # Z Z^T's own sums are over |Z| |Z|^T, not |Z Z^T|: N rounded products of size max|Z|^2 each
    bound = np.finfo(float).eps * (terms + N + 4) * (np.abs(dense) + np.max(np.diag(dense)) * (dense != 0)) @ np.abs(V)
    assert np.all(np.abs(got - dense @ V) <= bound + 1e-320)


@pytest.mark.parametrize("case", [(1, 129, 0, 32, 0, 1), (2, 257, 1, 40, 0, 0), (3, 50, 1, 9, 0, 1)])
def test_a_value_that_is_not_finite_stays_with_the_rows_it_couples_to(case):
    print("[case] not finite", case, file=sys.stderr, flush=True)
    P, dense, L = problem(case)
    V = np.random.default_rng(5).standard_normal((P.n, 20))
    want = ie.cov_apply(P, torch.from_numpy(V).cuda(), ie.default_opts()).cpu().numpy()
    spots = {3: (0, np.nan), 11: (P.n - 1, np.inf), 18: (P.n // 2, -np.inf)}
    for b, (r, v) in spots.items():
        V[r, b] = v
    got = ie.cov_apply(P, torch.from_numpy(V).cuda(), ie.default_opts()).cpu().numpy()
    for b in range(20):
        hit = L[:, spots[b][0]] != 0 if b in spots else np.zeros(P.n, bool)
        assert not np.isfinite(got[hit, b]).any()
        assert np.array_equal(got[~hit, b], want[~hit, b])
