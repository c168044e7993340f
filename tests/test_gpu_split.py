"""The split half-sweep (one field, the eight hops of a site in eight
wavefronts of a 64-site block) against the FP64 oracle and against the batched
kernel, at the sizes where its tiles, slabs and rules change.

Tolerances are those of test_gpu_parity.py: the normwise bounds of the storage
precision and the per-site bound derived there; a batch runs the lane-per-site
kernel, whose numbers the split kernel has to give bit for bit.
"""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import SITE_BOUND, THETA, THETA_GEN, dev, host, rel, site_err, tmq  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# one partial tile; two whole ones; slabs of one and two planes (z, t) with
# tiles that end inside a row; the last and the first 16-bit sizes of the rule
EDGES = [(2, 2, 2, 2), (4, 4, 4, 4), (10, 10, 4, 6), (12, 18, 6, 14), (32, 16, 12, 16), (32, 16, 14, 16)]


@pytest.mark.parametrize("theta", [THETA, THETA_GEN], ids=["t", "all"])
@pytest.mark.parametrize("variant", [0, 1, 3])
@pytest.mark.parametrize("dims", EDGES, ids=lambda d: "x".join(map(str, d)))
def test_split_half_sweep(tmq, dims, variant, theta, monkeypatch):  # noqa: F811
    monkeypatch.setenv("TMQ_HOP_VARIANT", str(variant))
    U = synth.random_gauge(dims, seed=301)
    lat = tmq.Lattice(dims)  # a lattice of its own: the forced variant is read at creation
    lat.load_gauge(U)
    psi = synth.gaussian_odd(dims, seed=31)
    p = tmq.params(0.1632, 0.004, theta)
    ref = oracle.Qhat(U, psi, 0.1632, 0.004, +1, theta)
    for prec, tol in (("fp64", 1e-13), ("fp32", 2e-6), ("fp16", 3e-3), ("bf16", 2.5e-2)):
        got = host(lat.apply_Qhat(p, +1, dev(psi), prec=prec))
        assert rel(got, ref) < tol and site_err(got, ref) < SITE_BOUND[prec], (prec, rel(got, ref))
    # every epilogue of a solve (norms, CG update, true residual), alone (split) and in a batch
    bs = [dev(psi), dev(synth.gaussian_odd(dims, seed=32))]
    ps = [p, tmq.params(0.16, 0.011, theta)]
    for sloppy in ("fp64", "fp32", "fp16"):
        opts = tmq.solver_opts(tol=1e-9, sloppy=sloppy, sloppy_link="fp32" if sloppy == "fp32" else "fp16")
        xs, infos = lat.solve_batch(ps, bs, opts)
        for i in range(2):
            x, info = lat.solve(ps[i], bs[i], opts)
            assert info.status == 0 and info.iters == infos[i].iters
            assert torch.equal(x, xs[i]), (sloppy, i)
    lat.close()


@pytest.mark.parametrize("dims", EDGES[:4], ids=lambda d: "x".join(map(str, d)))
def test_split_other_site_terms(tmq, dims):  # noqa: F811
    """The epilogues of the full-lattice operator and of M^-1, and links that are not SU(3)."""
    U = synth.random_gauge(dims, seed=302)
    V = int(np.prod(dims))
    lat = tmq.Lattice(dims)
    psi = synth.gaussian_spinor(dims + (4, 3), seed=33)
    p = tmq.params(0.15, 0.02, THETA_GEN)
    for links in (U, 1.02 * U):
        lat.load_gauge(links)
        for sign in (+1, -1):
            got = host(lat.apply_Q_full(p, sign, dev(psi.reshape(V, 4, 3))))
            ref = oracle.Q(links, psi, 0.15, 0.02, sign, THETA_GEN).reshape(V, 4, 3)
            assert rel(got, ref) < 1e-13 and site_err(got, ref) < SITE_BOUND["fp64"]
    lat.load_gauge(U)
    x, info = lat.solve_M(p, +1, dev(psi.reshape(V, 4, 3)), tmq.solver_opts(tol=1e-10))
    back = oracle.M(U, host(x).reshape(dims + (4, 3)), 0.15, 0.02, +1, THETA_GEN)
    assert info.status == 0 and rel(back, psi) < 2e-10
    lat.close()


@pytest.mark.parametrize("dims", [(4, 4, 4, 8), (2, 10, 4, 6), (8, 4, 4, 8)], ids=lambda d: "x".join(map(str, d)))
def test_small_full_cg(tmq, dims, monkeypatch):  # noqa: F811
    """The one-launch CG of tiny lattices over several blocks (two parities in
    one tile, a partial last tile, the largest size), and the way back to plain
    launches when its blocks give up waiting for each other (bounded wait of no
    ticks: every block leaves at once)."""
    V = int(np.prod(dims))
    U = synth.random_gauge(dims, seed=303)
    lat = tmq.Lattice(dims)
    lat.load_gauge(U)
    b = synth.gaussian_spinor(dims + (4, 3), seed=34).reshape(-1, 4, 3)
    p = tmq.params(0.16, 0.01, THETA_GEN)
    for opts in (tmq.solver_opts(tol=1e-10), tmq.solver_opts(tol=1e-13)):
        x, info = lat.solve_full(p, dev(b), opts)
        res = oracle.true_residual(U, b, host(x), 0.16, 0.01, THETA_GEN, eo=False)
        assert info.status == 0 and res <= opts.tol and abs(res - info.true_rel_residual) <= 1e-2 * res
        monkeypatch.setenv("TMQ_SMALL_CG_SPIN", "-1")
        x2, info2 = lat.solve_full(p, dev(b), opts)
        monkeypatch.delenv("TMQ_SMALL_CG_SPIN")
        assert info2.status == 0 and abs(info2.iters - info.iters) <= 2
        assert oracle.true_residual(U, b, host(x2), 0.16, 0.01, THETA_GEN, eo=False) <= opts.tol
    lat.close()


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (10, 10, 4, 6), (32, 16, 8, 16), (32, 16, 8, 18)],
                         ids=lambda d: "x".join(map(str, d)))
def test_canonical_buffers_in_place(tmq, dims):  # noqa: F811
    """Half-sweeps that read and write the caller's buffers: sizes on both sides
    of the rule (32 K sites), the operators in place, and the reduced
    precisions' results equal to the values their storage holds."""
    V = int(np.prod(dims))
    U = synth.random_gauge(dims, seed=304)
    lat = tmq.Lattice(dims)
    lat.load_gauge(U)
    p = tmq.params(0.1632, 0.004, THETA)
    psi = dev(synth.gaussian_odd(dims, seed=35))
    full = dev(synth.gaussian_spinor(dims + (4, 3), seed=36).reshape(V, 4, 3))
    for prec in ("fp64", "fp32", "fp16", "bf16"):
        out = lat.apply_Qhat(p, -1, psi, prec=prec)
        ref = oracle.Qhat(U, host(psi), 0.1632, 0.004, -1, THETA)
        assert rel(host(out), ref) < {"fp64": 1e-13, "fp32": 2e-6, "fp16": 3e-3, "bf16": 2.5e-2}[prec]
        v = psi.clone()
        lat.apply_Qhat(p, -1, v, out=v, prec=prec)
        assert torch.equal(v, out), prec
        if prec in ("fp16", "bf16"):
            codes, scale = lat.encode(out, prec)  # stored values encode to themselves
            dt = torch.float16 if prec == "fp16" else torch.bfloat16
            back = codes.view(dt).float() * scale[:, None]
            assert torch.equal(back.double(), torch.view_as_real(out).reshape(-1, 24))
        elif prec == "fp32":
            assert torch.equal(torch.view_as_real(out).float().double(), torch.view_as_real(out))
    out = lat.apply_QhatQhat(p, psi)
    assert rel(host(out), oracle.QhatQhat(U, host(psi), 0.1632, 0.004, THETA)) < 1e-13
    v = psi.clone()
    lat.apply_QhatQhat(p, v, out=v)
    assert torch.equal(v, out)
    out = lat.apply_Q_full(p, +1, full)
    assert rel(host(out), oracle.Q(U, host(full).reshape(dims + (4, 3)), 0.1632, 0.004, +1, THETA).reshape(V, 4, 3)) < 1e-13
    v = full.clone()
    lat.apply_Q_full(p, +1, v, out=v)
    assert torch.equal(v, out)
    lat.close()


@pytest.mark.parametrize("variant", [0, 1, 3])
@pytest.mark.parametrize("dims", EDGES[:4], ids=lambda d: "x".join(map(str, d)))
def test_split_doublet(tmq, dims, variant, monkeypatch):  # noqa: F811
    """One FP64 or FP32 doublet runs the split kernel, a batch the lane pairs:
    the operator against the oracle, and solves of both inner precisions (and of
    16-bit ones, whose true residual is the split FP64 kernel's) equal in a
    batch and alone."""
    monkeypatch.setenv("TMQ_HOP_VARIANT", str(variant))
    U = synth.random_gauge(dims, seed=305)
    lat = tmq.Lattice(dims)
    lat.load_gauge(U)
    V = int(np.prod(dims))
    bs = [dev(synth.gaussian_spinor((2, V // 2, 4, 3), seed=37 + i)) for i in range(2)]
    ps = [tmq.nd_params(0.15, 0.11, 0.09, THETA_GEN), tmq.nd_params(0.14, 0.05, 0.12, THETA_GEN)]
    ref = oracle.Qhat_nd(U, host(bs[0]), 0.15, 0.11, 0.09, +1, THETA_GEN)
    for prec, tol in (("fp64", 1e-13), ("fp32", 2e-6)):
        got = host(lat.apply_Qhat_nd(ps[0], +1, bs[0], prec=prec))
        assert rel(got, ref) < tol and site_err(got, ref) < SITE_BOUND[prec], (prec, rel(got, ref))
    for sloppy in ("fp64", "fp32", "fp16"):
        opts = tmq.solver_opts(tol=1e-9, sloppy=sloppy, sloppy_link="fp32" if sloppy == "fp32" else "fp16")
        xs, infos = lat.solve_nd_batch(ps, bs, opts)
        for i in range(2):
            x, info = lat.solve_nd(ps[i], bs[i], opts)
            assert info.status == 0 and info.iters == infos[i].iters and torch.equal(x, xs[i]), (sloppy, i)
    lat.close()


@pytest.mark.parametrize("sign", [+1, -1])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 2, 10), (8, 4, 4, 6)], ids=lambda d: "x".join(map(str, d)))
def test_solve_M_batch_passes(tmq, dims, sign):  # noqa: F811
    """Batched inversions with a zero source among them (its solution is zero,
    whatever the work fields held before), sources left as they were, and every
    tolerance met by the oracle's M: also the loose one, which a solve of the
    normal equations to the same tolerance often misses at this mass, so that
    correction rounds run."""
    U = synth.random_gauge(dims, seed=303)
    lat = tmq.Lattice(dims)
    lat.load_gauge(U)
    V = int(np.prod(dims))
    e = np.zeros((V, 4, 3), np.complex128)
    e[V // 2 + 1, 2, 1] = 1.0
    phis = [synth.gaussian_spinor(dims + (4, 3), seed=61).reshape(V, 4, 3), np.zeros_like(e), e]
    p = tmq.params(0.1632, 0.004, THETA)
    for tol in (1e-10, 1e-3):
        srcs = [dev(f) for f in phis]
        psis, infos = lat.solve_M_batch(p, sign, srcs, tmq.solver_opts(tol=tol, sloppy="fp16", sloppy_link="fp16"))
        for f, s, x, i in zip(phis, srcs, psis, infos):
            assert np.array_equal(host(s), f)
            if not f.any():
                assert not host(x).any() and i.status == 0
                continue
            full = f.reshape(dims + (4, 3))
            r = full - oracle.M(U, host(x).reshape(full.shape), 0.1632, 0.004, sign, THETA)
            res = float(np.linalg.norm(r) / np.linalg.norm(f))
            assert i.status == 0 and res <= tol * (1 + 1e-6), (tol, res)
            assert abs(res - i.true_rel_residual) <= 1e-3 * res + 1e-16
    lat.close()


@pytest.mark.parametrize("kappa", [0.1632, 1e160], ids=["", "overflow"])
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (16, 16, 16, 64), (16, 16, 16, 66)], ids=lambda d: "x".join(map(str, d)))
def test_alpha_in_the_half_sweep(tmq, dims, kappa):  # noqa: F811
    """One field forms alpha in its CG half-sweep up to 512 blocks (the second
    size has them, the third more), a batch in the scalar kernel: the same
    iterates bit for bit, and the same end where <p, A p> overflows."""
    U = synth.random_gauge((4, 4, 4, 4), seed=304)
    U = np.tile(U, tuple(-(-d // 4) for d in dims) + (1, 1, 1))[tuple(slice(d) for d in dims)]
    lat = tmq.Lattice(dims)
    lat.load_gauge(dev(np.ascontiguousarray(U)))
    n = int(np.prod(dims)) // 2
    gen = torch.Generator(device="cuda")
    gen.manual_seed(71)
    bs = [torch.view_as_complex(torch.randn(n, 4, 3, 2, dtype=torch.float64, device="cuda", generator=gen)) for _ in "ab"]
    p = tmq.params(kappa, 0.004, THETA)
    for prec in ("fp64", "fp32"):
        o = tmq.solver_opts(tol=1e-12, sloppy=prec, sloppy_link="fp32", max_iter=6)
        xs, infos = lat.solve_batch([p, p], bs, o, check=False)
        x1, i1 = lat.solve(p, bs[0], o, check=False)
        assert (i1.status, i1.iters) == (infos[0].status, infos[0].iters)
        assert (i1.iters == 6) == (kappa < 1)
        assert torch.equal(torch.view_as_real(x1).nan_to_num(7.0), torch.view_as_real(xs[0]).nan_to_num(7.0))
    lat.close()
