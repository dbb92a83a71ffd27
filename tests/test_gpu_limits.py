"""Calls at the limits of their options: iteration caps, the static workspace, the memory budget."""

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _B():
    import paper_1612_04846_amd as B
    return B


def _coeff(n, dim=2):
    return 1.0 + 0.5 * np.random.default_rng(n).random((n + 2,) * dim)


@pytest.mark.parametrize("cap", [2 ** 31 - 1, 2 ** 31 - 2, 1])
@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
def test_largest_iteration_cap(cap, prec):
    """The largest caps an int holds are no caps; a cap of 1 ends every solve
    after one iteration."""
    B = _B()
    n = 31
    kw = dict(weights=[1.0], shifts=[0.01], coeff=_coeff(n), precision=getattr(B, "BURA_" + prec), tol=1e-8)
    f = torch.from_numpy(synth.normal_rhs(n, 2, nrhs=1, tag=1011)).cuda()
    want = B.Plan(2, n, **kw).solve(f)
    print(f"cap {cap} {prec}", flush=True)
    plan = B.Plan(2, n, max_iter=cap, max_outer=1 if cap == 1 else 12, **kw)
    got = plan.solve(f, ok=(B.BURA_ENOCONV,) if cap == 1 else (B.BURA_OK,))
    if cap == 1:
        assert got.report.iters[0] == 1
    else:
        assert got.report.iters[0] == want.report.iters[0]
        assert torch.equal(got.u, want.u)
    plan.close()
