"""The coarse solve's workgroups: 256, 512 or 1024 threads by the points of its first level.

First coarse levels of 6^3, 15^2 and 16^2 points run 256 threads, 7^3, 22^2
and 8^3 512, larger ones 1024; 23^2 to 31^2 two points per thread of 512 where
at least 1024 systems share the launch.  A point's arithmetic is the same in
all of them, so a right-hand side's result is the same, bit for bit, in a wide
launch as alone.  Bound of a single solve: sum_j |c_j| tol |f| / s_j (1.1 for
the residual that FP64 plans update recursively).
"""

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n,R", [(3, 13, 3), (2, 31, 3), (2, 33, 3), (3, 15, 3), (2, 45, 3), (3, 17, 3),
                                     (2, 47, 400), (2, 63, 350), (2, 61, 342)])
@pytest.mark.parametrize("var", [False, True])
@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
def test_threads_of_the_coarse_solve(dim, n, R, var, prec):
    import paper_1612_04846_amd as B
    from oracle import operators, shifted, spectral
    tol, w, s = 1e-10, [0.5, 0.3, 0.2], [0.05, 0.4, 2.0]
    F = synth.normal_rhs(n, dim, nrhs=R, tag=1061)
    kw = dict(precision=getattr(B, "BURA_" + prec), tol=tol, weights=w, shifts=s)
    pick = [0, R - 1]
    if var:
        a = 1.0 + 0.5 * np.random.default_rng(n).random((n + 2,) * dim)
        A, _ = operators.scaled_operator(n, dim, a)
        ref = shifted.bura_by_solves(A, w, [-v for v in s], F[pick], method="direct")
        kw["coeff"] = a
    else:
        ref = spectral.bura_spectral(F[pick], dim, w, [-v for v in s])
        kw["omega"] = 0.8
    print(f"coarse threads: {dim}D {n} x {R} var={var} {prec}", flush=True)
    f = torch.from_numpy(F).cuda()
    many = B.Plan(dim, n, nrhs_max=R, **kw)
    res = many.solve(f)
    assert min(list(res.report.iters)[:3]) >= 1
    bound = 1.1 * tol * sum(c / v for c, v in zip(w, s)) * np.linalg.norm(F[pick].reshape(2, -1), axis=1)
    assert np.all(np.linalg.norm((res.u[pick].cpu().numpy() - ref).reshape(2, -1), axis=1) <= bound)
    one = B.Plan(dim, n, nrhs_max=1, **kw)
    for r in pick:
        assert torch.equal(one.solve(f[r:r + 1]).u[0], res.u[r])
    many.close()
    one.close()
