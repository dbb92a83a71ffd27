"""Solves whose output overlaps their input.

A solve reads its right-hand sides for the last time before it writes u, so u
may be f, or share any part of its memory.  The direct solution writes u in
the pass of its residual test unless the two overlap; the systems that it
leaves over their tolerance form their residual from f.

Both solves of a comparison do the same operations on every system; the
combine may run in another kernel, which adds the same terms in the same
order.  Rounding can differ by the contraction of a product and a sum, at most
2^-53 of every partial sum: (terms + 1) 2^-53 sum_j |w_j x_j|, with the sum at
most 100 |u| for the terms below (checked on the host for white noise): 1e-13.
"""

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _B():
    import paper_1612_04846_amd as B
    return B


def _rel(a, b):
    a, b = a.cpu().numpy(), b.cpu().numpy()
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _terms(B):
    c, d, _ = B.bura_coefficients(0.5, 5)
    return c, [-x for x in d]


@pytest.mark.parametrize("dim,n", [(2, 63), (2, 511), (3, 31)])
@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
def test_slot_solve_with_a_loose_tolerance(dim, n, prec):
    """Right-hand side 0 iterates from zero (a tolerance of 1e-4), 1 is solved
    directly; 511^2 is large enough for the combine to join the residual test."""
    B = _B()
    w, s = _terms(B)
    f = torch.from_numpy(synth.normal_rhs(n, dim, nrhs=2, tag=1001)).cuda()
    h = B.bura_plan_create_slots(dim, n, 6, B.bura_opts_default(nrhs_max=3, precision=getattr(B, "BURA_" + prec)))
    print(f"in place: slots {dim}D {n} {prec}", flush=True)
    want = torch.empty_like(f)
    rep = B.bura_solve_slots(h, 6, f, want, [(w, s)] * 2, tols=[1e-4, 1e-10])
    assert max(list(rep.iters)[:6]) >= 1
    B.bura_solve_slots(h, 6, f, f, [(w, s)] * 2, tols=[1e-4, 1e-10])
    assert _rel(f, want) <= 1e-13
    B.bura_plan_destroy(h)


# forms of plan, each with a tolerance that the direct solution meets (1e-10)
# and one under its rounding, 0.3 of the largest residual that it reports
# (an FP64 plan's recursive residual goes on to fall)
FORMS = ["single", "per-pole", "multi", "multistep", "product", "beta2", "variable"]


@pytest.mark.parametrize("n", [63, 511])
@pytest.mark.parametrize("tight", [False, True])
@pytest.mark.parametrize("form", FORMS)
def test_plan_solved_in_place(form, n, tight):
    B = _B()
    args = dict(alpha=0.5, k=7)
    if form == "per-pole":
        args.update(schedule=B.BURA_PER_POLE)
    elif form == "multi":
        args.update(alpha=[0.25, 0.5, 0.75], k=[7, 5, 9])
    elif form == "multistep":
        args.update(alpha=[0.5, 0.25], k=[7, 6], form="multistep")
    elif form == "product":
        args.update(alpha=0.5, k=5, form="product")
    elif form == "beta2":
        args.update(alpha=0.5, k=4, beta=2)
    elif form == "variable":
        args.update(coeff=1.0 + 0.5 * np.random.default_rng(3).random((n + 2, n + 2)))
    f = torch.from_numpy(synth.normal_rhs(n, 2, nrhs=1, tag=1002)).cuda()
    tol = 1e-10
    if tight:
        plan = B.Plan(2, n, **args, precision=B.BURA_FP64, tol=tol)
        tol = 0.3 * max(plan.solve(f).report.relres)
        plan.close()
    print(f"in place: {form} n={n} tol={tol:.1e}", flush=True)
    plan = B.Plan(2, n, **args, precision=B.BURA_FP64, tol=tol)
    res = plan.solve(f)
    want = res.u.reshape(-1)
    if tight or form == "variable":
        assert max(res.report.iters) >= 1
    N = n * n
    # the input is the whole output (one output), each of its parts, and a
    # range that starts one value into it
    for at in sorted({0, want.numel() - N, 1}):
        buf = torch.zeros(want.numel() + 1, dtype=torch.float64, device="cuda")
        buf[at:at + N] = f.reshape(-1)
        plan.solve(buf[at:at + N].view(1, n, n), buf[:want.numel()].view(res.u.shape))
        # two solves to a tolerance: the bound of either is far below 1e-9 for
        # white noise; the same operations give rounding
        assert _rel(buf[:want.numel()], want) <= 1e-13
    plan.close()


def test_submitted_in_place():
    B = _B()
    w, s = _terms(B)
    n = 63
    f = torch.from_numpy(synth.normal_rhs(n, 2, nrhs=1, tag=1003)).cuda()
    h = B.bura_plan_create_slots(2, n, 6, B.bura_opts_default(nrhs_max=1))
    want = torch.empty_like(f)
    B.bura_solve_slots(h, 6, f, want, [(w, s)], tols=[1e-5])
    torch.cuda.synchronize()
    code, _ = B.bura_wait(B.bura_submit_slots(h, 6, f, f, [(w, s)], tols=[1e-5]))
    assert code == B.BURA_OK
    assert _rel(f, want) <= 1e-13
    B.bura_plan_destroy(h)
