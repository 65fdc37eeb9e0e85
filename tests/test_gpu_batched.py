"""Batched instances (infoesrf_update_batched) through the C ABI.

On the pool of streams every instance of a batch must give exactly the bits of
the same instance run alone: instances share no arithmetic, each keeps its own
workspace slice, and the per-system work does not depend on which stream or host
thread issued it.  In one persistent launch over every instance the systems run
on another workgroup shape (four rows a thread), which sums the dots in another
order: there each member agrees with the single-instance call to 1e-7 and each
system's iteration count within 2.  Instances are also checked against the FP64
oracle (each member to 1e-6, the FP64-mode bound at rtol 1e-8).
"""
import sys

import numpy as np
import pytest

import synthetic as syn
from parity import upd  # noqa: E402
from oracle import infoesrf_ref as ref

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2503_00253_amd import infoesrf as ie  # noqa: E402


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def layered_problem(seed):
    """4 x 50 layered grid, every 2nd site of every layer observed."""
    rng = np.random.default_rng(seed)
    nz, nx, N = 4, 50, 6
    n = nz * nx
    X = rng.standard_normal((n, N)) + 0.5 * np.sin(np.arange(n) / 7.0)[:, None]
    bz, bx, table = syn.gc_table_2d(3.0, 1.0)
    idx = np.array([z * nx + x for z in range(nz) for x in range(0, nx, 2)], dtype=np.int32)
    m = idx.size
    return syn.Problem(n=n, N=N, m=m, X=np.asfortranarray(X), h_ptr=np.arange(m + 1, dtype=np.int32), h_idx=idx,
                       h_w=1.0 + 0.25 * np.cos(np.arange(m)), r_var=0.3 * (1.0 + 0.5 * rng.random(m)),
                       y=rng.standard_normal(m), nz=nz, nx=nx, periodic_z=0, periodic_x=1, bz=bz, bx=bx,
                       table=table, truth=np.zeros(n), Q=5, ell=100.0, name="layered-4x50")


def batch():
    return [
        syn.gaussian_problem(512, 16, 20.0, 12.0, 4, 0.25, 6, 100.0, 101, name="g512"),
        syn.config1(),
        layered_problem(13),
        syn.gaussian_problem(1024, 12, 40.0, 30.0, 4, 0.5, 5, 1000.0, 103, name="g1024"),
        syn.gaussian_problem(256, 8, 10.0, 20.0, 4, 0.25, 3, 100.0, 102, name="g256"),
    ]


def run_single(P, prob, s, p, opts):
    Xa, st = ie.perturbation_update(P, s, p, opts)
    mu, sm = ie.mean_update(P, prob.y, opts)
    return Xa.cpu().numpy(), mu.cpu().numpy(), st, sm


def make_opts(domain, precision, P=None, **kw):
    if domain == "lattice":
        kw.update(apply_domain=ie.DOMAIN_OBS_LATTICE)
        if P is not None:
            kw.update(lattice=P.lattice())
    return ie.default_opts(precision=precision, **kw)


@pytest.mark.parametrize("domain,precision,tail", [("state", ie.FP64, 0), ("lattice", ie.FP64, 100000),
                                                   ("lattice", ie.MIXED_BF16, 0), ("lattice", ie.MIXED_FP32, 0)])
def test_batched_equals_single_instances(domain, precision, tail):
    """Every instance of the batched call equals the single-instance call bit for bit, with the
    batched call's default hand-over to the persistent kernel (the last 64 systems) or with every
    system handed over after the first step."""
    probs = batch()
    Ps = [ie.Problem.from_synthetic(pr) for pr in probs]
    nodes = [ie.quadrature_elliptic(pr.Q, pr.ell) for pr in probs]
    lats = [P.lattice() for P in Ps] if domain == "lattice" else None
    say("batched", domain, precision, tail, [pr.name for pr in probs])
    runner = ie.BatchedRunner(Ps, nodes, make_opts(domain, precision, tail_systems=tail), ys=[pr.y for pr in probs],
                              lattices=lats)
    code = runner.run()
    torch.cuda.synchronize()
    assert code == ie.OK
    one = runner.one_launch()
    say("  one launch:", one)
    Xs, mus = runner.results()
    st = runner.stats(code)
    off = 0
    totals = np.zeros(ie.NUM_COUNTERS, dtype=np.int64)
    # per-system iterations of the two schedules (one persistent launch against the batched loop
    # handing over at 64 live systems): with FP32 inner applies the first sweep runs to 1e-7 of the
    # residual, near the FP32 apply's rounding level, so where each schedule's recursive residual
    # crosses it moves by a few iterations
    it_tol = 4 if precision == ie.MIXED_FP32 else 2
    for j, (pr, P, (s, p)) in enumerate(zip(probs, Ps, nodes)):
        say("single", j, pr.name)
        Xa, mu, s1, sm = run_single(P, pr, s, p, make_opts(domain, precision, P, tail_systems=tail or 64))
        S = len(s) * pr.N
        if one:
            assert upd(Xs[j].cpu().numpy(), Xa) < 1e-7, (j, pr.name)
            assert upd(mus[j].cpu().numpy(), mu) < 1e-7
            assert np.max(np.abs(st.iters[off:off + S] - s1.iters)) <= it_tol
            assert abs(int(st.iters[off + S]) - int(sm.iters[0])) <= it_tol
        else:
            assert np.array_equal(Xs[j].cpu().numpy(), Xa), (j, pr.name)
            assert np.array_equal(mus[j].cpu().numpy(), mu), (j, pr.name)
            assert np.array_equal(st.iters[off:off + S], s1.iters)
            assert np.array_equal(st.relres[off:off + S], s1.relres)
            assert st.iters[off + S] == sm.iters[0] and st.relres[off + S] == sm.relres[0]
        totals += s1.counters + sm.counters
        off += S + 1
    assert off == len(st.iters)
    assert st.converged.all()
    if not one:
        for c in (ie.CNT_APPLIES, ie.CNT_ITERATIONS, ie.CNT_SWEEPS, ie.CNT_NOT_CONVERGED):
            assert st.counter(c) == totals[c], c
    else:
        assert st.counter(ie.CNT_NOT_CONVERGED) == 0
        assert st.counter(ie.CNT_ITERATIONS) == int(st.iters.sum())
    assert st.counter(ie.CNT_STATUS) == 0


@pytest.mark.parametrize("count", [1, 2, 256, 300])
def test_queue_of_many_instances(count):
    """The queue of one persistent launch takes in every instance's systems whatever their number
    (below, at and over the 256 threads that add up the earlier instances' counts): copies of three
    problems give the same bits wherever they stand in the batch, and agree with the oracle."""
    kinds = [syn.gaussian_problem(n, N, 5.0, 8.0, 2, 0.25, 3, 100.0, 300 + n, name="q%d" % n)
             for n, N in ((64, 4), (48, 3), (96, 5))]
    Ps = [ie.Problem.from_synthetic(kinds[j % 3]) for j in range(count)]
    lats = [P.lattice() for P in Ps]
    nodes = [ie.quadrature_elliptic(3, 100.0)] * count
    say("queue of", count)
    runner = ie.BatchedRunner(Ps, nodes, make_opts("lattice", ie.FP64, tail_systems=100000),
                              ys=[kinds[j % 3].y for j in range(count)], lattices=lats)
    code = runner.run()
    torch.cuda.synchronize()
    assert code == ie.OK
    assert count < 2 or runner.one_launch()
    assert runner.stats(code).converged.all()
    Xs, mus = runner.results()
    for j in range(count):
        assert torch.equal(Xs[j], Xs[j % 3]) and torch.equal(mus[j], mus[j % 3]), j
    for j in range(min(3, count)):
        pr = kinds[j]
        s0, p0, _ = ref.quadrature_elliptic(pr.Q, pr.ell)
        want = np.sqrt(pr.N - 1) * ref.perturbation_update_quadrature(ref.DenseProblem.from_problem(pr), s0, p0)
        assert upd(Xs[j].cpu().numpy(), want) < 1e-6, pr.name


@pytest.mark.parametrize("precision", [ie.FP64, ie.MIXED_FP32])
@pytest.mark.parametrize("m,c", [(1025, 8.0), (1026, 9.0), (1160, 10.0), (1535, 11.0), (1537, 8.5), (2047, 9.5),
                                 (2048, 10.5)])
def test_four_rows_a_thread(m, c, precision):
    """Systems of 1024 < m <= 2048 observations in the persistent kernel, alone and in a batch: odd
    and even m at the ends of its wavefronts' second pairs, stencils (2 ceil(2 c) - 1 points) of every
    remainder of a quad and of a chunk of two; against the state-domain FP64 loop, another path
    altogether, at 1e-6, the FP64-mode bound at rtol 1e-8."""
    prob = syn.gaussian_problem(4 * m, 4, 24.0, 4 * c, 4, 0.25, 3, 100.0, 41, name="four-%d" % m)
    say("four rows", m, c, precision)
    P = ie.Problem.from_synthetic(prob)
    nodes = ie.quadrature_elliptic(prob.Q, prob.ell)
    Xr, mr, _, _ = run_single(P, prob, *nodes, ie.default_opts())
    opts = make_opts("lattice", precision, P, n_ritz=4, oversample=4, tail_systems=100000)
    Xa, mu, st, sm = run_single(P, prob, *nodes, opts)
    assert st.converged.all() and sm.converged.all()
    mean = prob.X.mean(axis=1)
    assert upd(Xa, Xr) < 1e-6 and upd(mu - mean, mr - mean) < 1e-6
    runner = ie.BatchedRunner([P, P], [nodes, nodes], opts, ys=[prob.y, prob.y], lattices=[P.lattice()] * 2)
    assert runner.run() == ie.OK
    torch.cuda.synchronize()
    Xs, mus = runner.results()
    assert runner.one_launch()
    for j in range(2):
        assert upd(Xs[j].cpu().numpy(), Xr) < 1e-6 and upd(mus[j].cpu().numpy() - mean, mr - mean) < 1e-6


def test_batched_instance_matches_oracle():
    probs = batch()
    Ps = [ie.Problem.from_synthetic(pr) for pr in probs]
    nodes = [ie.quadrature_elliptic(pr.Q, pr.ell) for pr in probs]
    say("batched vs oracle")
    runner = ie.BatchedRunner(Ps, nodes, ie.default_opts(), ys=[pr.y for pr in probs])
    runner.run()
    torch.cuda.synchronize()
    Xs, mus = runner.results()
    for j in (1, 2):
        pr = probs[j]
        dp = ref.DenseProblem.from_problem(pr)
        s0, p0, _ = ref.quadrature_elliptic(pr.Q, pr.ell)
        want = np.sqrt(pr.N - 1) * ref.perturbation_update_quadrature(dp, s0, p0)
        got = Xs[j].cpu().numpy()
        assert upd(got, want) < 1e-6, pr.name
        mwant = ref.mean_update_cholesky(dp, pr.y)
        assert upd(mus[j].cpu().numpy() - dp.mu, mwant - dp.mu) < 1e-6


def test_batched_without_host_sync_matches():
    probs = batch()
    Ps = [ie.Problem.from_synthetic(pr) for pr in probs]
    nodes = [ie.quadrature_elliptic(pr.Q, pr.ell) for pr in probs]
    lats = [P.lattice() for P in Ps]
    say("batched host_sync 0")
    base = ie.BatchedRunner(Ps, nodes, make_opts("lattice", ie.MIXED_BF16, max_iter=200),
                            ys=[pr.y for pr in probs], lattices=lats)
    base.run()
    torch.cuda.synchronize()
    nosync = ie.BatchedRunner(Ps, nodes, make_opts("lattice", ie.MIXED_BF16, max_iter=200, host_sync=0),
                              ys=[pr.y for pr in probs], lattices=lats)
    assert nosync.run() == ie.OK
    torch.cuda.synchronize()
    st = nosync.stats()
    assert st.counter(ie.CNT_STATUS) == 0 and st.counter(ie.CNT_NOT_CONVERGED) == 0
    (xa, ma), (xb, mb) = base.results(), nosync.results()
    for j in range(len(probs)):
        assert np.array_equal(xa[j].cpu().numpy(), xb[j].cpu().numpy()), j
        assert np.array_equal(ma[j].cpu().numpy(), mb[j].cpu().numpy()), j


def test_batched_reports_failing_instance():
    probs = batch()
    probs[3].r_var = probs[3].r_var.copy()
    probs[3].r_var[7] = -1.0   # detected on the device by the input checks
    Ps = [ie.Problem.from_synthetic(pr) for pr in probs]
    nodes = [ie.quadrature_elliptic(pr.Q, pr.ell) for pr in probs]
    say("batched failing instance")
    runner = ie.BatchedRunner(Ps, nodes, ie.default_opts(), ys=[pr.y for pr in probs])
    with pytest.raises(ie.InfoEsrfError) as e:
        runner.run()
    torch.cuda.synchronize()
    assert e.value.code == ie.ERR_INVALID_ARG and "instance 3" in str(e.value)
    Xs, _ = runner.results()
    # the other instances are still solved
    Xa, _ = ie.perturbation_update(Ps[0], *nodes[0], ie.default_opts())
    if runner.one_launch():
        assert upd(Xs[0].cpu().numpy(), Xa.cpu().numpy()) < 1e-7
    else:
        assert np.array_equal(Xs[0].cpu().numpy(), Xa.cpu().numpy())


def test_full_size_uneven_batch_matches_oracle():
    """The 64-instance uneven batch (n = 4 U{128..2048}, N in {16, 32, 48, 64}, Q = U{8..24}) in
    one batched call with the benchmark's options (FP64, observed lattice); three instances against
    the dense oracle, each member to 1e-6: the largest n, the largest n among those with N = 64,
    and the largest Q."""
    probs = syn.config4_instances()
    Ps = [ie.Problem.from_synthetic(pr) for pr in probs]
    nodes = [ref.quadrature_elliptic(pr.Q, pr.ell)[:2] for pr in probs]
    say("uneven batch of 64, full size")
    runner = ie.BatchedRunner(Ps, nodes, ie.default_opts(apply_domain=ie.DOMAIN_OBS_LATTICE),
                              ys=[pr.y for pr in probs], lattices=[P.lattice() for P in Ps])
    code = runner.run()
    torch.cuda.synchronize()
    assert code == ie.OK
    st = runner.stats(code)
    assert st.converged.all() and np.all(st.relres <= 1e-8)
    Xs, mus = runner.results()
    largest_n = max(range(len(probs)), key=lambda j: probs[j].n)
    largest_n64 = max((j for j in range(len(probs)) if probs[j].N == 64), key=lambda j: probs[j].n)
    largest_q = max(range(len(probs)), key=lambda j: (probs[j].Q, probs[j].n))
    for j in sorted({largest_n, largest_n64, largest_q}):
        pr = probs[j]
        say("  instance", j, "n", pr.n, "N", pr.N, "Q", pr.Q)
        dp = ref.DenseProblem.from_problem(pr)
        s0, p0 = nodes[j]
        want = np.sqrt(pr.N - 1) * ref.perturbation_update_quadrature(dp, s0, p0)
        err = upd(Xs[j].cpu().numpy(), want)
        merr = upd(mus[j].cpu().numpy() - dp.mu, ref.mean_update_eig(dp, pr.y) - dp.mu)
        say("    members", err, "mean", merr)
        assert err < 1e-6 and merr < 1e-6


@pytest.mark.parametrize("precision", [ie.FP64, ie.MIXED_FP32])
def test_one_launch_graph_and_host_sync(precision):
    """The one-launch batch without host synchronization equals the host-synchronized call bit for
    bit, and so do HIP-graph replays of it (three replays, each checked, with eager work between)."""
    probs = batch()
    Ps = [ie.Problem.from_synthetic(pr) for pr in probs]
    nodes = [ie.quadrature_elliptic(pr.Q, pr.ell) for pr in probs]
    lats = [P.lattice() for P in Ps]
    say("one launch: host sync vs none vs graph", precision)
    base = ie.BatchedRunner(Ps, nodes, make_opts("lattice", precision), ys=[pr.y for pr in probs], lattices=lats)
    assert base.one_launch()
    assert base.run() == ie.OK
    torch.cuda.synchronize()
    xa, ma = base.results()
    want = [x.clone() for x in xa]
    wmean = [m.clone() for m in ma]
    nosync = ie.BatchedRunner(Ps, nodes, make_opts("lattice", precision, host_sync=0), ys=[pr.y for pr in probs],
                              lattices=lats)
    assert nosync.one_launch()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        nosync.run()   # eager (sets kernel attributes before capture)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    st = nosync.stats()
    assert st.counter(ie.CNT_STATUS) == 0 and st.counter(ie.CNT_NOT_CONVERGED) == 0
    xb, mb = nosync.results()
    for j in range(len(probs)):
        assert torch.equal(xb[j], want[j]) and torch.equal(mb[j], wmean[j]), j
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        nosync.run()
    for rep in range(3):
        for x in xb:
            x.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        xg, mg = nosync.results()
        for j in range(len(probs)):
            assert torch.equal(xg[j], want[j]) and torch.equal(mg[j], wmean[j]), (rep, j)
