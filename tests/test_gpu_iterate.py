"""The multigrid iteration of constant-coefficient plans, which their solves
otherwise leave to the direct solution: with the damping set (omega) a plan
iterates from zero, and the counts of every solve here show that it did.

Tolerances: system j stops at a residual of at most tol |f|, so an output is
off by at most sum_j |c_j| tol |f| / (lambda_min + s_j) (1.1 for the residual
that FP64 plans update recursively); two solves differ by twice that.  A
V-cycle takes the same iterations up to rounding whichever kernels run it:
counts agree within one.
"""

import numpy as np
import pytest

import synth
from conftest import oracle_coeffs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

OMEGA = {2: 0.8, 3: 6.0 / 7.0}


def _B():
    import paper_1612_04846_amd as B
    return B


def _bound(dim, n, b, tol, F):
    lam = np.sin(np.pi / (2 * (n + 1))) ** 2   # the smallest eigenvalue of the scaled operator
    amp = sum(abs(c) / (lam - d) for c, d in zip(b.c_f64, b.d_f64))
    return 1.1 * tol * amp * np.linalg.norm(F.reshape(F.shape[0], -1), axis=1)


def _solve(B, dim, n, b, F, prec, tol, **kw):
    plan = B.Plan(dim, n, weights=b.c_f64, shifts=[-x for x in b.d_f64], precision=getattr(B, "BURA_" + prec),
                  nrhs_max=F.shape[0], tol=tol, omega=OMEGA[dim], **kw)
    res = plan.solve(torch.from_numpy(F).cuda())
    torch.cuda.synchronize()
    nt = len(b.c_f64)
    out = res.u.cpu().numpy(), list(res.report.iters)[:nt], list(res.report.outer)[:nt]
    plan.close()
    assert min(out[1]) >= 1
    return out


def _off(u, ref):
    return np.linalg.norm((u - ref).reshape(u.shape[0], -1), axis=1)


# 63 -> 31 -> 15 (31 coarse columns of 32, 31 coarse rows of 8), 127 (four
# coarse rows of tiles, a segment of 16 coarse planes and a short one), 47 (an
# even coarsest level), 191 and 95 (workgroups of 128 columns over a ragged
# second tile, of 64 below), one and two sweeps
LEVELS3 = [(63, "FP64", 2), (63, "MIXED", 2), (127, "MIXED", 2), (47, "MIXED", 2), (63, "MIXED", 1), (31, "FP64", 1),
           (95, "FP64", 2), (191, "MIXED", 2), (191, "FP64", 1)]


@pytest.mark.parametrize("n,prec,nu", LEVELS3)
def test_3d_level_kernels_fused_separate_and_unfused(n, prec, nu):
    from oracle import spectral
    B = _B()
    b = oracle_coeffs(0.75, 7) if n < 100 else oracle_coeffs(0.5, 5)
    tol = 1e-11
    F = synth.normal_rhs(n, 3, nrhs=2 if n < 150 else 1, tag=1031)
    ref = spectral.bura_spectral(F, 3, b.c_f64, b.d_f64)
    bound = _bound(3, n, b, tol, F)
    counts = []
    for v in (0, B.BURA_VARIANT_NO_FOLDXR, B.BURA_VARIANT_UNFUSED):
        print(f"3D levels: n={n} {prec} nu={nu} variant={v}", flush=True)
        u, it, _ = _solve(B, 3, n, b, F, prec, tol, nu_pre=nu, nu_post=nu, variant=v)
        assert np.all(_off(u, ref) <= bound)
        counts.append(it)
    for it in counts[1:]:
        assert all(abs(x - y) <= 1 for x, y in zip(counts[0], it))


@pytest.mark.parametrize("dim,n,prec,unfused", [(2, 255, "FP64", False), (2, 255, "MIXED", False),
                                                (2, 127, "MIXED", True), (2, 127, "FP64", True),
                                                (3, 63, "MIXED", True)])
def test_folded_vector_updates_and_a_separate_pass(dim, n, prec, unfused):
    """x += alpha p deferred into the stencil product, r -= alpha q in the first
    pre-smoothing kernel, several systems converging at different iterations."""
    from oracle import spectral
    B = _B()
    b = oracle_coeffs(0.75, 9)
    tol = 1e-11
    F = synth.normal_rhs(n, dim, nrhs=2, tag=1032)
    ref = spectral.bura_spectral(F, dim, b.c_f64, b.d_f64)
    v = B.BURA_VARIANT_UNFUSED if unfused else 0
    out = []
    for w in (v, v | B.BURA_VARIANT_NO_FOLDXR):
        print(f"folded updates: {dim}D {n} {prec} variant={w}", flush=True)
        u, it, _ = _solve(B, dim, n, b, F, prec, tol, variant=w)
        assert np.all(_off(u, ref) <= _bound(dim, n, b, tol, F))
        out.append(it)
    assert len(set(out[0])) > 1
    assert all(abs(x - y) <= 1 for x, y in zip(*out))


@pytest.mark.parametrize("variant", ["", "NO_FOLDXR"])
def test_wide_refinement_updates_x64_in_the_residual_pass(variant):
    """512 systems of 255^2: x64 += e in the pass of the FP64 residual, the first
    update assigning x64; row-marching kernels by default, tiles below.  A zero
    right-hand side reads 0, and a narrow launch (two separate passes) agrees."""
    from oracle import spectral
    B = _B()
    n, R, tol = 255, 64, 1e-11
    b = oracle_coeffs(0.5, 7)
    F = synth.normal_rhs(n, 2, nrhs=R, tag=1033)
    F[5] = 0.0
    ref = spectral.bura_spectral(F, 2, b.c_f64, b.d_f64)
    bound = _bound(2, n, b, tol, F)
    kw = dict(variant=getattr(B, "BURA_VARIANT_" + variant) if variant else 0)
    print(f"wide refinement {variant}", flush=True)
    u, _, outer = _solve(B, 2, n, b, F, "MIXED", tol, **kw)
    assert min(outer) >= 2
    assert np.all(u[5] == 0.0)
    assert np.all(_off(u, ref) <= bound)
    un, _, _ = _solve(B, 2, n, b, F[:4], "MIXED", tol, **kw)
    assert np.all(_off(un, u[:4]) <= 2 * bound[:4])


# Systems that the direct solution leaves over their tolerance go on from its
# result.  FP64 slot solves at 1e-4 iterate from x = 0 there: the residual in
# tiles (63^2, 30^2), in rows (255^2 and enough systems) and in 3D.
@pytest.mark.parametrize("dim,n,R", [(2, 63, 2), (2, 30, 3), (2, 255, 40), (3, 31, 2), (3, 63, 1)])
@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
def test_slots_that_go_on_iterating(dim, n, R, prec):
    from oracle import spectral
    B = _B()
    b = oracle_coeffs(0.5, 5)
    w, s = b.c_f64, [-x for x in b.d_f64]
    F = synth.normal_rhs(n, dim, nrhs=R, tag=1034)
    ref = spectral.bura_spectral(F, dim, b.c_f64, b.d_f64)
    tols = [1e-4 if r % 2 == 0 else 1e-10 for r in range(R)]
    print(f"slots go on: {dim}D {n} x {R} {prec}", flush=True)
    f = torch.from_numpy(F).cuda()
    u = torch.empty_like(f)
    h = B.bura_plan_create_slots(dim, n, 7, B.bura_opts_default(nrhs_max=R + 1, precision=getattr(B, "BURA_" + prec)))
    rep = B.bura_solve_slots(h, 7, f, u, [(w, s)] * R, tols=tols)
    B.bura_plan_destroy(h)
    assert min(list(rep.iters)[:6]) >= 1
    off, bound = _off(u.cpu().numpy(), ref), _bound(dim, n, b, 1.0, F)
    assert np.all(off <= bound * tols)
    assert np.all((off <= 1e-9 * np.linalg.norm(ref.reshape(R, -1), axis=1))[1::2])


GO_ON = [(2, 63, "single"), (2, 255, "single"), (2, 200, "single"), (3, 31, "single"), (2, 127, "per-pole"),
         (2, 127, "multi"), (2, 127, "multistep"), (2, 127, "product"), (2, 127, "beta2")]


@pytest.mark.parametrize("dim,n,form", GO_ON)
@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
def test_plans_that_go_on_from_the_direct_solution(dim, n, form, prec):
    """A tolerance of half the largest residual that the direct solution of a
    smooth right-hand side leaves: the systems over it iterate on from there (a
    mixed plan's refinement may be at the rounding of its FP64 residual already
    and end at its limit of steps: BURA_ENOCONV, with the result no worse)."""
    B = _B()
    args = dict(alpha=0.5, k=7)
    if form == "per-pole":
        args.update(schedule=B.BURA_PER_POLE)
    elif form == "multi":
        args.update(alpha=[0.25, 0.75], k=[7, 9])
    elif form == "multistep":
        args.update(alpha=[0.5, 0.25], k=[7, 6], form="multistep")
    elif form == "product":
        args.update(alpha=0.5, k=6, form="product")
    elif form == "beta2":
        args.update(alpha=0.5, k=4, beta=2)
    p = getattr(B, "BURA_" + prec)
    x = np.arange(1, n + 1) / (n + 1)
    g = np.meshgrid(*([x] * dim), indexing="ij")
    f = torch.from_numpy(np.prod([1.0 + q * (1.0 - q) for q in g], axis=0)[None].copy()).cuda()
    first = B.Plan(dim, n, precision=p, tol=1e-10, **args)
    a = first.solve(f)
    nt = a.report.nterms
    res = np.array(list(a.report.relres)[:nt])
    tol = 0.5 * float(res.max())
    print(f"go on: {dim}D {n} {form} {prec} direct residual {res.max():.1e}", flush=True)
    plan = B.Plan(dim, n, precision=p, tol=tol, **args)
    c = plan.solve(f, ok=(B.BURA_OK, B.BURA_ENOCONV) if prec == "MIXED" else (B.BURA_OK,))
    its = np.array(list(c.report.iters)[:nt])
    print(f"  iterations {its.tolist()}, residual {max(list(c.report.relres)[:nt]):.1e}", flush=True)
    assert its.max() >= 1
    if prec == "FP64" or c.report.status == B.BURA_OK:
        assert max(list(c.report.relres)[:nt]) <= tol
    else:
        assert max(list(c.report.relres)[:nt]) <= float(res.max())
    # each is within its residual over lambda_min of the exact result, and the
    # smooth right-hand side's output is no shorter than the right-hand side
    lam = 0.9 * (np.pi / 2) ** 2 / (n + 1) ** 2
    for u, v in zip(a.u.reshape(-1, n ** dim), c.u.reshape(-1, n ** dim)):
        assert float((u - v).norm()) <= 4.0 * (res.max() / lam) * float(u.norm())
    again = plan.solve(f, ok=(B.BURA_OK, B.BURA_ENOCONV))
    assert torch.equal(again.u, c.u)
    first.close()
    plan.close()
