"""Solves that end at their iteration limit: TMQ_ENOCONV leaves the last iterate
of the CG, compared with the oracle's FP64 iterate of that number, and a limit
of just the iterations that a solve needs changes nothing about it.

Tolerances, relative to |x_k|: in FP64 k applications of A and the sums round
at 1e-13 each; in a reduced precision an application of A is two of Qhat, which
test_gpu_parity.py bounds by 2e-6 (FP32) and 3e-3 (FP16), and its error enters
alpha, x and the next p: five such applications per iteration are allowed.  An
update of x left out, or done twice, is an error of a tenth to 1 here.
"""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import THETA, THETA_GEN, dev, host, rel, tmq  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

KAPPA, MUT = 0.1632, 0.01
# inner precision, link precision, mode, iterations looked at, tolerance per iteration
MODES = {
    "fp64": ("fp64", "fp32", 0, (1, 2, 3, 6), 1e-12),
    "fp32": ("fp32", "fp32", 0, (1, 2, 3, 6), 5 * 4e-6),
    "fp16": ("fp16", "fp16", 0, (1, 2), 5 * 6e-3),
    "switch": ("fp32", "fp32", 1, (1, 2, 3, 6), 1e-12),
}


def options(t, mode, **kw):
    sloppy, link, m, _, _ = MODES[mode]
    return t.solver_opts(tol=1e-10, sloppy=sloppy, sloppy_link=link, mode=m, **kw)


@pytest.mark.parametrize("mode", MODES)
def test_last_iterate_at_the_limit(tmq, mode):  # noqa: F811
    dims = (6, 4, 2, 10)
    U = synth.random_gauge(dims, seed=401)
    lat = tmq.Lattice(dims)
    lat.load_gauge(U)
    bs = [synth.gaussian_odd(dims, seed=41 + i) for i in range(2)]
    muts = [MUT, 0.03]
    ps = [tmq.params(KAPPA, m, THETA_GEN) for m in muts]
    for k in MODES[mode][3]:
        o = options(tmq, mode, max_iter=k)
        xs, infos = lat.solve_batch(ps, [dev(b) for b in bs], o, check=False)
        x1, i1 = lat.solve(ps[0], dev(bs[0]), o, check=False)
        assert torch.equal(x1, xs[0]) and i1.iters == infos[0].iters
        for b, m, x, i in zip(bs, muts, xs, infos):
            want, _ = oracle.cg(U, b, KAPPA, m, THETA_GEN, max_iter=k)
            assert i.status == tmq.TMQ_ENOCONV and i.iters == k
            assert rel(host(x), want) < k * MODES[mode][4], (k, rel(host(x), want))
    lat.close()


@pytest.mark.parametrize("mode", ["fp64", "fp32", "fp16"])
def test_last_iterate_of_a_doublet(tmq, mode):  # noqa: F811
    dims = (4, 4, 4, 6)
    U = synth.random_gauge(dims, seed=402)
    lat = tmq.Lattice(dims)
    lat.load_gauge(U)
    nd = (0.17, 0.1105, 0.0935)
    bs = [synth.gaussian_spinor((2, int(np.prod(dims)) // 2, 4, 3), seed=43 + i) for i in range(2)]
    p = tmq.nd_params(*nd, THETA_GEN)
    for k in MODES[mode][3]:
        o = options(tmq, mode, max_iter=k)
        xs, infos = lat.solve_nd_batch([p, p], [dev(b) for b in bs], o, check=False)
        x1, i1 = lat.solve_nd(p, dev(bs[0]), o, check=False)
        assert torch.equal(x1, xs[0]) and i1.iters == infos[0].iters
        for b, x, i in zip(bs, xs, infos):
            want, _ = oracle.cg_nd(U, b, *nd, THETA_GEN, max_iter=k)
            assert i.status == tmq.TMQ_ENOCONV and i.iters == k
            assert rel(host(x), want) < k * MODES[mode][4], (k, rel(host(x), want))
    lat.close()


@pytest.mark.parametrize("mode", MODES)
def test_limit_of_the_iterations_needed(tmq, mode):  # noqa: F811
    dims = (8, 4, 4, 6)
    U = synth.random_gauge(dims, seed=403)
    lat = tmq.Lattice(dims)
    lat.load_gauge(U)
    b = dev(synth.gaussian_odd(dims, seed=45))
    p = tmq.params(KAPPA, MUT, THETA)
    x, info = lat.solve(p, b, options(tmq, mode))
    assert info.status == 0
    x2, info2 = lat.solve(p, b, options(tmq, mode, max_iter=info.iters), check=False)
    assert (info2.status, info2.iters, info2.reliable_updates) == (0, info.iters, info.reliable_updates)
    assert torch.equal(x, x2) and info2.true_rel_residual == info.true_rel_residual
    lat.close()


def test_served_requests_with_limits_of_their_own(tmq):  # noqa: F811
    """Requests that end at different limits, and one that converges, share an engine."""
    dims = (8, 4, 4, 6)
    U = synth.random_gauge(dims, seed=404)
    p = tmq.params(KAPPA, MUT, THETA)
    limits = [1, 3, 0, 2, 6]
    bs = [synth.gaussian_odd(dims, seed=46 + i) for i in range(len(limits))]
    for mode in ("fp64", "fp32"):
        with tmq.Server(max_batch=8) as srv:
            lid = srv.add_lattice(dims, dev(U))
            ts = [srv.submit(lid, p, dev(b), options(tmq, mode, max_iter=k)) for b, k in zip(bs, limits)]
            got = [srv.wait(t, timeout=60) for t in ts]
        for (x, i), b, k in zip(got, bs, limits):
            if k == 0:
                assert i.status == 0 and oracle.true_residual(U, b, host(x), KAPPA, MUT, THETA) <= 1e-10
                continue
            want, _ = oracle.cg(U, b, KAPPA, MUT, THETA, max_iter=k)
            assert i.status == tmq.TMQ_ENOCONV and i.iters == k
            assert rel(host(x), want) < k * MODES[mode][4], (mode, k, rel(host(x), want))
