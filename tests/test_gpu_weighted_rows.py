"""Observation rows of many entries on the GPU: the row sums a workgroup, a wavefront or a thread each,
the CSC copy, the dense S and diag(S) by tiles, at the edges of their chunks (2 and 16 entries, a
wavefront, one and several tiles, rows past the tiled kernel's 256), against the FP64 oracle.

The converged update agrees to 1e-6, the FP64-mode bound at rtol 1e-8.
"""
import sys

import numpy as np
import pytest

import synthetic as syn
from parity import upd
from oracle import infoesrf_ref as ref

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2503_00253_amd import infoesrf as ie  # noqa: E402


def weighted(n, m, entries, N, seed, bad=None):
    """m rows whose lengths run over `entries`, smooth positive weights around spread centres."""
    base = syn.gaussian_problem(n, N, 6.0, 9.0, n // m, 0.25, 4, 100.0, seed, name="w%d" % n)
    rng = np.random.default_rng(seed)
    ptr, idx, w = [0], [], []
    for k in range(m):
        cnt = entries[k % len(entries)]
        j = np.sort((k * n // m + np.arange(cnt) - cnt // 2) % n)
        idx.append(j)
        w.append((0.5 + rng.random(cnt)) / cnt)
        ptr.append(ptr[-1] + cnt)
    return syn.Problem(n=n, N=N, m=m, X=base.X, h_ptr=np.array(ptr, np.int32),
                       h_idx=np.concatenate(idx).astype(np.int32), h_w=np.concatenate(w), r_var=np.full(m, 0.3),
                       y=rng.standard_normal(m), nz=1, nx=n, periodic_z=0, periodic_x=1, bz=0, bx=base.bx,
                       table=base.table, truth=np.zeros(n), Q=4, ell=100.0, name="rows-%d" % n)


@pytest.mark.parametrize("entries", [(1, 2, 3), (15, 16, 17), (31, 33, 64), (65, 130, 177), (255, 256, 257, 300)])
@pytest.mark.parametrize("N", [3, 13, 24])
def test_rows_of_many_entries_match_oracle(entries, N):
    print("[case] rows", entries, N, file=sys.stderr, flush=True)
    prob = weighted(600, 30, entries, N, 7 + N)
    P = ie.Problem.from_synthetic(prob)
    dp = ref.DenseProblem.from_problem(prob)
    s, p, _ = ref.quadrature_elliptic(prob.Q, prob.ell)
    want = np.sqrt(N - 1) * ref.perturbation_update_quadrature(dp, s, p)
    for kw in ({}, {"n_ritz": 4, "oversample": 4}):
        Xa, st = ie.perturbation_update(P, *ie.quadrature_elliptic(prob.Q, prob.ell), ie.default_opts(**kw))
        assert st.converged.all()
        assert upd(Xa.cpu().numpy(), want) < 1e-6
        mu, sm = ie.mean_update(P, prob.y, ie.default_opts(**kw))
        assert upd(mu.cpu().numpy() - dp.mu, ref.mean_update_eig(dp, prob.y) - dp.mu) < 1e-6
