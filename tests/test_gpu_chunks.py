"""The ways a PCG solve advances: watched by the host at every iteration, in
captured chunks of iterations, or in chunks of eager launches.

The iterations are the same launches on the same data, so results and counts
are bitwise equal; a system that has converged inside a chunk is left alone by
the rest of it.  Even grids have no hierarchy and run in chunks by default;
grids with one run in chunks with folded scalar updates and while profiling.
"""

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _B():
    import paper_1612_04846_amd as B
    return B


def _solve(B, dim, n, prec, var, repeats=3, profile=False, **kw):
    """(u, iterations per term) of a solve repeated with other work of the
    caller's in between, checked to be the same every time."""
    coeff = 1.0 + 0.5 * np.random.default_rng(n).random((n + 2,) * dim) if var else None
    f = torch.from_numpy(synth.normal_rhs(n, dim, nrhs=2, tag=1021)).cuda()
    plan = B.Plan(dim, n, 0.5, 5, nrhs_max=3, precision=getattr(B, "BURA_" + prec), tol=1e-9, coeff=coeff,
                  **({} if var else dict(omega=0.8)), **kw)
    if profile:
        B.bura_plan_profile(plan.handle, 1)
    out = []
    for _ in range(repeats):
        res = plan.solve(f)
        other = (f * 2.0).sum()
        torch.cuda.synchronize()
        out.append((res.u, list(res.report.iters)[:6]))
        assert float(other) == float(other)
    plan.close()
    assert min(out[0][1]) >= 1
    for u, it in out[1:]:
        assert torch.equal(u, out[0][0]) and it == out[0][1]
    return out[0]


GRIDS = [(2, 64, True), (2, 63, True), (2, 63, False), (3, 24, True), (3, 31, False)]


@pytest.mark.parametrize("dim,n,var", GRIDS)
@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
def test_chunks_watched_and_eager_agree(dim, n, var, prec):
    B = _B()
    print(f"chunks: {dim}D {n} var={var} {prec}", flush=True)
    want, its = _solve(B, dim, n, prec, var)
    for check in (1, 3, 4, 7):
        for v in (0, B.BURA_VARIANT_NO_GRAPH, B.BURA_VARIANT_FOLD_SCALARS,
                  B.BURA_VARIANT_FOLD_SCALARS | B.BURA_VARIANT_NO_GRAPH):
            u, it = _solve(B, dim, n, prec, var, check_every=check, variant=v)
            assert it == its and torch.equal(u, want), (check, v)
    u, it = _solve(B, dim, n, prec, var, profile=True)
    assert it == its and torch.equal(u, want)


def test_large_grid_without_a_hierarchy_is_watched():
    """Six systems of 600^2 hold 2.2e6 points: watched, and the same solution
    as in chunks (one system at a time)."""
    B = _B()
    n = 600
    coeff = 1.0 + 0.5 * np.random.default_rng(n).random((n + 2, n + 2))
    f = torch.from_numpy(synth.normal_rhs(n, 2, nrhs=1, tag=1022)).cuda()
    out = []
    for schedule in (B.BURA_BATCHED, B.BURA_PER_POLE):
        plan = B.Plan(2, n, 0.5, 5, precision=B.BURA_FP64, tol=1e-8, coeff=coeff, schedule=schedule)
        res = plan.solve(f)
        out.append((res.u, list(res.report.iters)[:6]))
        plan.close()
    assert min(out[0][1]) >= 1 and out[0][1] == out[1][1]
    assert torch.equal(out[0][0], out[1][0])
