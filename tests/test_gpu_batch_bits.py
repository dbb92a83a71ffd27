"""A right-hand side's result does not depend on what else is in its solve.

The direct solution's tiles and transforms, and whether the combine joins the
residual test, go by the size of the launch; every value is summed in the same
order in all of them, so a batch and single solves agree bitwise.  The sizes
have the batch in 64 x 64 tiles (200, 40^3) or with the combine in the test's
pass (255, 511, 63^3) where a single solve has not.
"""

import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n,R", [(2, 200, 24), (2, 255, 7), (2, 511, 3), (2, 127, 20), (3, 40, 12), (3, 63, 5)])
@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
def test_batch_equals_single_solves(dim, n, R, prec):
    import paper_1612_04846_amd as B
    f = torch.from_numpy(synth.normal_rhs(n, dim, nrhs=R, tag=1051)).cuda()
    kw = dict(precision=getattr(B, "BURA_" + prec), tol=1e-10)
    print(f"batch bits: {dim}D {n} x {R} {prec}", flush=True)
    many, one = B.Plan(dim, n, 0.5, 7, nrhs_max=R, **kw), B.Plan(dim, n, 0.5, 7, nrhs_max=1, **kw)
    u = many.solve(f).u
    for r in (0, R // 2, R - 1):
        assert torch.equal(one.solve(f[r:r + 1]).u[0], u[r])
    # right-hand sides with their own terms, one at a loose tolerance
    c, d, _ = B.bura_coefficients(0.5, 5)
    terms = (c, [-x for x in d])
    tols = [1e-10] * R
    tols[R // 2] = 1e-5
    h = B.bura_plan_create_slots(dim, n, 6, B.bura_opts_default(nrhs_max=R, **kw))
    us = torch.empty_like(f)
    B.bura_solve_slots(h, 6, f, us, [terms] * R, tols=tols)
    for r in (0, R // 2, R - 1):
        alone = torch.empty_like(f[r:r + 1])
        B.bura_solve_slots(h, 6, f[r:r + 1].contiguous(), alone, [terms], tols=tols[r:r + 1])
        assert torch.equal(alone[0], us[r])
    B.bura_plan_destroy(h)
    many.close()
    one.close()
