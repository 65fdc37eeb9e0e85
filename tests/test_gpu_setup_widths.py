"""The preconditioner's setup at sketch widths on both sides of every change of its small kernels
(odd and even widths, 16 / 17 columns of the Gram kernels, 20 / 21 of the register Cholesky, 32 / 33 of the
eigensolver's blocks a thread, the widest), with a full and a deficient rank of S.

Against the FP64 oracle at 1e-6, the FP64-mode bound at rtol 1e-8; the preconditioner has to do its work:
with p Ritz pairs no system takes more iterations than without any.
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


@pytest.mark.parametrize("c", [8.0, 1000.0])  # localized; L = 1 nearly, so rank(S) about N - 1 = 9
@pytest.mark.parametrize("p,over", [(4, 5), (8, 8), (10, 7), (8, 11), (10, 10), (10, 11), (20, 12), (20, 13), (20, 28)])
def test_update_at_sketch_width(p, over, c):
    print("[case] width", p, over, c, file=sys.stderr, flush=True)
    prob = syn.gaussian_problem(480, 10, c, 12.0, 4, 0.25, 4, 100.0, 11, name="w480")
    P = ie.Problem.from_synthetic(prob)
    s0, p0, _ = ref.quadrature_elliptic(prob.Q, prob.ell)
    want = np.sqrt(prob.N - 1) * ref.perturbation_update_quadrature(ref.DenseProblem.from_problem(prob), s0, p0)
    s, w = ie.quadrature_elliptic(prob.Q, prob.ell)
    _, plain = ie.perturbation_update(P, s, w, ie.default_opts(n_ritz=0, oversample=0))
    for kw in ({}, {"apply_domain": ie.DOMAIN_OBS_LATTICE, "lattice": P.lattice()}):
        Xa, st = ie.perturbation_update(P, s, w, ie.default_opts(n_ritz=p, oversample=over, **kw))
        assert st.converged.all()
        assert upd(Xa.cpu().numpy(), want) < 1e-6
        assert np.max(st.iters) <= np.max(plain.iters)
