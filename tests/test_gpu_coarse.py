"""GPU parity of the multigrid iteration over the coarse solve's first levels.

The coarse levels are solved by one workgroup that holds 1, 2, 4 or 6 points
per thread: the sizes below put the first coarse level at the edges of those
ranges (31^2 and 9^3 in one point per thread, 38^2, 11^3 and 12^3 in two,
47^2, 63^2 and 15^3 in four, 72^2, 17^3 and 18^3 in six), with odd ones that
coarsen on and even ones (38, 72, 12, 18) that are the last level.  The 3D
sizes also run the level kernels that walk fewer planes per workgroup.
Constant coefficients run with the damping set, so that they iterate.

Tolerance: system j stops at a residual of at most tol |f|, so the output is
off by at most sum_j |c_j| tol |f| / (lambda_min + s_j) (every eigenvalue of
the variable operator is at least min a times the constant one's, over the
scaling); the oracle's own solves get a tenth of that.  A V(2,2) cycle takes
off about a digit or more, so tol = 1e-11 needs 11 iterations or so: at most 20.
"""

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [(2, n) for n in (63, 77, 95, 127, 145)] + [(3, n) for n in (19, 23, 25, 31, 35, 37)]


@pytest.mark.parametrize("dim,n", SIZES)
@pytest.mark.parametrize("coeff", ["const", "var"])
@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
def test_first_coarse_level_sizes(dim, n, coeff, prec):
    import paper_1612_04846_amd as B
    from oracle import operators, shifted, spectral
    tol, w, s = 1e-11, [0.4, 0.35, 0.25], [0.0, 0.02, 1.5]
    F = synth.normal_rhs(n, dim, nrhs=1, tag=970 + n)
    lam_min = 4.0 * dim * (n + 1) ** 2 * np.sin(np.pi / (2 * (n + 1))) ** 2
    kw = {}
    if coeff == "var":
        x = np.linspace(0.0, 1.0, n + 2)
        grids = np.meshgrid(*([x] * dim), indexing="ij")
        a = 1.0 + 0.5 * np.prod([np.sin(3.0 * g + 0.4 * i) for i, g in enumerate(grids)], axis=0)
        A, lam = operators.scaled_operator(n, dim, a)
        ref = shifted.bura_by_solves(A, w, [-v for v in s], F, method="direct" if dim == 2 else "cg")
        lam_min *= float(a.min()) / lam
        kw["coeff"] = a
    else:
        ref = spectral.bura_spectral(F, dim, w, [-v for v in s])
        lam_min /= 4.0 * dim * (n + 1) ** 2
        kw["omega"] = 0.8
    bound = 1.1 * tol * sum(c / (lam_min + v) for c, v in zip(w, s)) * np.linalg.norm(F)
    print(f"coarse: dim={dim} n={n} {coeff} {prec}", flush=True)
    plan = B.Plan(dim, n, weights=w, shifts=s, precision=getattr(B, "BURA_" + prec), tol=tol, **kw)
    res = plan.solve(torch.from_numpy(np.ascontiguousarray(F)).cuda())
    torch.cuda.synchronize()
    its = list(res.report.iters)[:3]
    err = float(np.linalg.norm(res.u.cpu().numpy() - ref))
    print(f"  iters {its}, error {err / np.linalg.norm(ref):.1e}, bound {bound / np.linalg.norm(ref):.1e}")
    assert max(its) <= 20 and its[0] >= 2
    assert err <= bound
    plan.close()


@pytest.mark.parametrize("n,nu,prec", [(1023, 3, "FP64"), (1023, 2, "FP64"), (1023, 3, "MIXED"), (767, 3, "FP64"),
                                       (511, 2, "MIXED")])
def test_row_kernels_at_their_widest(n, nu, prec):
    """The row-marching 2D kernels with as many columns as they take (three FP64
    sweeps need more than 64 KiB of LDS there); the bound of the test above,
    with constant coefficients: launch shapes that are set make a plan iterate."""
    import paper_1612_04846_amd as B
    from oracle import spectral
    tol, w, s = 1e-11, [0.5, 0.5], [0.02, 1.5]
    F = synth.normal_rhs(n, 2, nrhs=1, tag=980 + n)
    ref = spectral.bura_spectral(F, 2, w, [-v for v in s])
    bound = 1.1 * tol * sum(c / v for c, v in zip(w, s)) * np.linalg.norm(F)
    plan = B.Plan(2, n, weights=w, shifts=s, precision=getattr(B, "BURA_" + prec), tol=tol, nu_pre=nu, nu_post=nu)
    f = torch.from_numpy(np.ascontiguousarray(F)).cuda()
    for v in (3, 4):
        print(f"rows: n={n} nu={nu} {prec} variant {v}", flush=True)
        plan.tiles = [v] * len(plan.tiles)
        res = plan.solve(f)
        torch.cuda.synchronize()
        its = list(res.report.iters)[:2]
        assert 1 <= max(its) <= 20
        assert float(np.linalg.norm(res.u.cpu().numpy() - ref)) <= bound
    plan.close()
