"""Calls at the limits of their options: iteration caps, the static workspace, the memory budget, tuning."""

import time

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


# The systems of one grid that the 64 MiB workspace has always taken: grids
# whose coarsest level had no exact solve before the coarse solve took more
# LDS (121^2, 145^2, 149^2; 29^3, 37^3: with the hierarchy they would need one
# vector a system more) and small 3D grids (where the direct solution's partial
# sums outnumber the other kernels').
STATIC = [(2, 121, "FP64", 81), (2, 145, "FP64", 56), (2, 149, "MIXED", 83), (3, 7, "FP64", 3392),
          (3, 7, "MIXED", 5277), (3, 13, "MIXED", 828), (3, 19, "MIXED", 265), (3, 29, "FP64", 49),
          (3, 37, "FP64", 23), (3, 37, "MIXED", 36)]


@pytest.mark.parametrize("dim,n,prec,nsys", STATIC)
def test_static_workspace_takes_as_many_systems(dim, n, prec, nsys):
    from oracle import spectral
    B = _B()
    tol, shift = 1e-8, 0.5
    F = synth.normal_rhs(n, dim, nrhs=nsys, tag=1012)
    f = torch.from_numpy(F.reshape(nsys, -1)).cuda()
    u = torch.empty_like(f)
    print(f"static: {dim}D {n} {prec} {nsys} systems", flush=True)
    o = B.bura_opts_default(precision=getattr(B, "BURA_" + prec), nrhs_max=nsys, tol=tol)
    B.bura_solve_static(dim, n, [1.0], [shift], f, u, o)
    ref = spectral.bura_spectral(F[-2:], dim, [1.0], [-shift]).reshape(2, -1)
    # |(A + s)^-1 r| <= tol |f| / s
    d = np.linalg.norm(u[-2:].cpu().numpy() - ref, axis=1)
    assert np.all(d <= 1.1 * tol / shift * np.linalg.norm(F[-2:].reshape(2, -1), axis=1))
    over = B.bura_opts_default(nrhs_max=2 * nsys, tol=tol)
    f2 = torch.zeros((2 * nsys, n ** dim), dtype=torch.float64, device="cuda")
    rep = B.bura_solve_static(dim, n, [1.0], [shift], f2, torch.empty_like(f2), over, ok=(B.BURA_ETOOBIG,))
    assert rep.status == B.BURA_ETOOBIG


def _smallest_budget(B, dim, n, var, prec):
    lo, hi = 0, 1 << 30
    while hi - lo > 4096:
        m = (lo + hi) // 2
        try:
            B.Plan(dim, n, weights=[1.0] * 2, shifts=[0.1, 0.5], coeff=_coeff(n, dim) if var else None,
                   precision=getattr(B, "BURA_" + prec), hbm_budget=m).close()
            hi = m
        except B.BuraError as e:
            assert e.code == B.BURA_ENOMEM
            lo = m
    return hi


@pytest.mark.parametrize("dim,n,prec", [(2, 121, "FP64"), (2, 149, "MIXED"), (3, 29, "FP64"), (3, 37, "MIXED")])
@pytest.mark.parametrize("var", [False, True])
def test_budget_that_was_enough_without_a_hierarchy(dim, n, prec, var):
    """The hierarchy of a grid whose coarse solve needs the larger LDS is given
    up where it does not fit the budget: such a grid asks for no more than the
    next one, which is even and has none, and the same vectors per point.  (The
    coarser levels' face weights are counted all the same: 1/3 of the finest
    level's in 2D, 1/7 in 3D; 64 KiB for partial sums, which go by blocks.)"""
    B = _B()
    print(f"budget: {dim}D {n} {prec} var={var}", flush=True)
    a, b = (_smallest_budget(B, dim, m, var, prec) for m in (n, n + 1))
    faces = dim * (n + 2) ** dim * 12 / (2 ** dim - 1) if var else 0
    assert a <= b * (n / (n + 1)) ** dim + faces + 65536
    # and such a plan solves
    kw = dict(weights=[1.0] * 2, shifts=[0.1, 0.5], coeff=_coeff(n, dim) if var else None,
              precision=getattr(B, "BURA_" + prec), tol=1e-9, omega=0.8)
    f = torch.from_numpy(synth.normal_rhs(n, dim, nrhs=1, tag=1013)).cuda()
    small, full = B.Plan(dim, n, hbm_budget=a, **kw), B.Plan(dim, n, **kw)
    us, uf = small.solve(f), full.solve(f)
    assert max(us.report.iters) > 2 * max(uf.report.iters)
    d = float((us.u - uf.u).norm())
    assert d <= 2.2e-9 * (1 / 0.1 + 1 / 0.5) * float(f.norm())
    small.close()
    full.close()


def test_autotune_times_constant_coefficient_plans():
    """A plan that the direct solution starts iterates all the same where a
    tolerance is loose, or a residual over it: autotune = 1 times its kernels.
    Creation then holds a warm-up and three timings of at least four variants
    of three kernels, more than 30 solves by iteration; counted as ten."""
    B = _B()
    n = 223
    f = torch.from_numpy(synth.normal_rhs(n, 2, nrhs=3, tag=1014)).cuda()
    kw = dict(alpha=0.5, k=7, nrhs_max=3, tol=1e-10)
    it = B.Plan(2, n, omega=0.8, **kw)
    solve = []
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        it.solve(f)
        solve.append(time.perf_counter() - t)
    torch.cuda.synchronize()
    t = time.perf_counter()
    tuned = B.Plan(2, n, autotune=1, **kw)
    t = time.perf_counter() - t
    print(f"iterated solve {min(solve) * 1e3:.2f} ms, creation {t * 1e3:.1f} ms, tiles {tuned.tiles}")
    assert t >= 10 * min(solve)
    assert all(0 <= v < B.BURA_TILE_VARIANTS for v in tuned.tiles)
    res = tuned.solve(f)
    assert max(res.report.iters) == 0   # and its own solves still start from the direct solution
    for p in (it, tuned):
        p.close()
