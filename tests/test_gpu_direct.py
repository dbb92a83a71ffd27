"""GPU parity of the direct solution that starts constant-coefficient solves.

Plans with constant coefficients and the library's own damping form every
shifted system's solution in the sine basis first (two transforms per axis:
products on the FP64 matrix cores, or fast Fourier transforms where n + 1 is
a power of two), test its FP64 residual and iterate only from there.
The sizes sit at the edges of the 32- and 64-wide tiles and of the halves the
transforms split into (odd sizes have an unpaired middle value), with one
right-hand side (32 x 32 tiles) and with enough of them for 64 x 64 ones.

Tolerance: a transform sums n products, so its rounding error is at most
n 2^-53 of the vector per axis and direction, and the random signs of the
errors keep the smooth coefficients' amplification from adding to that for
the random right-hand sides used here: 16 dim n 2^-53 covers the 2 dim
transforms and the oracle's own rounding (n >= 16 in the formula).
"""

import numpy as np
import pytest

import synth
from conftest import oracle_coeffs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _B():
    import paper_1612_04846_amd as B
    return B


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _rel(u, ref):
    nb = ref.shape[0]
    a, b = u.reshape(nb, -1), ref.reshape(nb, -1)
    return float(np.max(np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)))


SIZES = [(2, n, 1) for n in (1, 2, 3, 16, 31, 32, 33, 63, 64, 65, 127, 128, 129)]
SIZES += [(3, n, 1) for n in (1, 2, 5, 16, 17, 31, 33, 64, 65)]
SIZES += [(2, 65, 64), (2, 130, 24), (3, 31, 8)]   # 64 x 64 tiles
# fast Fourier transforms (n + 1 = 2^p; 63 and 127 are above), each length
SIZES += [(2, 255, 3), (2, 511, 2), (2, 1023, 1), (2, 2047, 1), (3, 63, 2), (3, 127, 1)]


@pytest.mark.parametrize("dim,n,nrhs", SIZES)
@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
def test_direct_solution_matches_oracle(dim, n, nrhs, prec):
    from oracle import spectral
    B = _B()
    alpha, k = 0.5, 5
    b = oracle_coeffs(alpha, k)
    F = synth.normal_rhs(n, dim, nrhs=nrhs, tag=900 + n)
    print(f"direct: dim={dim} n={n} nrhs={nrhs} {prec}", flush=True)
    plan = B.Plan(dim, n, weights=b.c_f64, shifts=[-x for x in b.d_f64], nrhs_max=nrhs,
                  precision=getattr(B, "BURA_" + prec), tol=1e-10)
    res = plan.solve(_dev(F))
    err = _rel(_host(res.u), spectral.bura_spectral(F, dim, b.c_f64, b.d_f64))
    print(f"  rel err {err:.2e}, relres {max(list(res.report.relres)[:k + 1]):.1e}")
    assert list(res.report.iters)[:k + 1] == [0] * (k + 1)   # no iteration was needed
    assert 0.0 <= max(list(res.report.relres)[:k + 1]) <= 1e-10
    assert err <= 16 * dim * max(n, 16) * 2.0 ** -53
    plan.close()


def _solve_form(B, form, F, **kw):
    """One solve of each form of plan on a 63^2 (63^3 for "3d") grid; returns (u, report)."""
    n, nr = F.shape[-1], F.shape[0]
    if form == "slots":
        pairs = [(0.5, 5), (0.3, 7), (0.75, 9)][:nr]
        terms = []
        for a, k in pairs:
            c, d, _ = B.bura_coefficients(a, k)
            terms.append((c, [-x for x in d]))
        h = B.bura_plan_create_slots(2, n, 12, B.bura_opts_default(nrhs_max=nr + 1, **kw))
        f, u = _dev(F), torch.empty(F.shape, dtype=torch.float64, device="cuda")
        rep = B.bura_solve_slots(h, 12, f, u, terms)
        out = _host(u)
        B.bura_plan_destroy(h)
        return out, rep
    if form == "static":
        b = oracle_coeffs(0.5, 5)
        f = _dev(F.reshape(nr, -1))
        u = torch.empty_like(f)
        rep = B.bura_solve_static(2, n, b.c_f64, [-x for x in b.d_f64], f, u, B.bura_opts_default(nrhs_max=nr, **kw))
        return _host(u).reshape(F.shape), rep
    dim, args = 2, dict(nrhs_max=nr)
    if form == "single":
        args.update(alpha=0.5, k=7)
    elif form == "3d":
        dim = 3
        args.update(alpha=0.25, k=6)
    elif form == "fewer":
        args.update(alpha=0.5, k=7, nrhs_max=nr + 2)
    elif form == "per-pole":
        args.update(alpha=0.5, k=7, schedule=B.BURA_PER_POLE, nrhs_max=nr + 1)
    elif form == "multi":
        args.update(alpha=[0.25, 0.75], k=[7, 9])
    elif form == "multistep":
        args.update(alpha=[0.5, 0.25], k=[7, 6], form="multistep", nrhs_max=nr + 1)
    elif form == "product":
        args.update(alpha=0.5, k=6, form="product")
    elif form == "beta2":
        args.update(alpha=0.5, k=4, beta=2)
    elif form == "sinc":
        args.update(alpha=0.5, kprime=B.sinc_kprime(0.5, 7))
    elif form == "unscaled":
        args.update(alpha=0.5, k=7, rhs_unscaled=1)
    plan = B.Plan(dim, n, **args, **kw)
    res = plan.solve(_dev(F))
    out = _host(res.u)
    plan.close()
    return out, res.report


FORMS = ["single", "3d", "fewer", "per-pole", "multi", "multistep", "product", "beta2", "sinc", "unscaled", "slots",
         "static"]


@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
@pytest.mark.parametrize("form", FORMS)
def test_every_form_agrees_with_the_multigrid_solution(form, prec):
    """The same plan with the damping set by the caller iterates from zero (as
    the iteration counts show); both solutions agree to the tolerance of the
    iterated one, 1e-12 in the residual of every system (1e-9 in u, the bound
    the iterated solutions are held to against the oracle)."""
    B = _B()
    dim = 3 if form == "3d" else 2
    F = synth.normal_rhs(63, dim, nrhs=2, tag=951)
    kw = dict(precision=getattr(B, "BURA_" + prec), tol=1e-12)
    print(f"form {form} {prec}", flush=True)
    u_dir, r_dir = _solve_form(B, form, F, **kw)
    u_mg, r_mg = _solve_form(B, form, F, omega=0.8, **kw)
    nt = r_dir.nterms
    print(f"  direct iters {list(r_dir.iters)[:nt]}, multigrid iters {list(r_mg.iters)[:nt]}")
    assert min(list(r_mg.iters)[:nt]) >= 1
    d = u_dir.reshape(-1, *F.shape), u_mg.reshape(-1, *F.shape)
    assert max(_rel(a, b) for a, b in zip(*d)) <= 1e-9


def test_loose_tolerances_zero_and_nan_in_one_slot_solve():
    """A slot solve mixes a right-hand side that starts from the direct
    solution, one whose tolerance (1e-4) leaves it to the iteration, one that
    is 0 and an unused slot; each result is the one of its own plan."""
    B = _B()
    n = 95
    F = synth.normal_rhs(n, 2, nrhs=3, tag=952)
    F[2] = 0.0
    c, d, _ = B.bura_coefficients(0.5, 5)
    s = [-x for x in d]
    h = B.bura_plan_create_slots(2, n, 8, B.bura_opts_default(nrhs_max=4, tol=1e-10))
    f = _dev(F)
    u = torch.full_like(f, 7.0)
    B.bura_solve_slots(h, 8, f, u, [(c, s)] * 3, tols=[1e-10, 1e-4, 1e-10])
    out = _host(u)
    B.bura_plan_destroy(h)
    for r, tol in ((0, 1e-10), (1, 1e-4)):
        plan = B.Plan(2, n, weights=c, shifts=s, tol=tol)
        res = plan.solve(_dev(F[r:r + 1]))
        assert (max(list(res.report.iters)[:6]) == 0) == (tol < 1e-6)
        one = _host(res.u)
        plan.close()
        if r == 0:
            assert np.array_equal(out[0], one[0])
        else:
            assert _rel(out[1:2], one) <= 1e-6
    assert np.all(out[2] == 0.0)
    # a non-finite right-hand side: its own status, the other one untouched
    plan = B.Plan(2, n, weights=c, shifts=s, nrhs_max=2, tol=1e-10)
    G = F[:2].copy()
    G[1, 5, 5] = np.inf
    res = plan.solve(_dev(G), ok=(B.BURA_ENAN,))
    u2 = _host(res.u)
    plan.close()
    assert res.report.status == B.BURA_ENAN
    assert np.array_equal(u2[0], out[0])


def test_multigrid_counts_agree_where_the_damping_is_set():
    """The fused 3D level kernels and the one-kernel-per-step V-cycle with two
    sweeps, on plans that iterate from zero: the same counts within one."""
    B = _B()
    F = _dev(synth.normal_rhs(63, 3, nrhs=1, tag=953))
    its = []
    for v in (0, B.BURA_VARIANT_UNFUSED):
        plan = B.Plan(3, 63, 0.5, 5, precision=B.BURA_MIXED, tol=1e-10, omega=6.0 / 7.0, variant=v)
        its.append(list(plan.solve(F).report.iters)[:6])
        plan.close()
    assert min(its[0]) >= 3 and all(abs(a - b) <= 1 for a, b in zip(*its))


# one workgroup ends the solve (the smallest; 1020 systems), a copy does (more
# systems; more partial sums), the general kernels start and end it (a pole at a time)
REPORTS = [(2, 1, 1, "BATCHED"), (2, 15, 170, "BATCHED"), (2, 15, 256, "BATCHED"), (3, 63, 20, "BATCHED"),
           (2, 255, 1, "BATCHED"), (2, 33, 3, "PER_POLE")]


@pytest.mark.parametrize("dim,n,nrhs,schedule", REPORTS)
def test_state_reaches_the_host_alike_on_every_way(dim, n, nrhs, schedule):
    """The report of a solve as the device writes it, and as it is copied (what
    a profiled solve does): the same solution, and sums that differ by the order
    of at most 32768 terms, 2^-38; with the caller's stream busy and idle."""
    B = _B()
    b = oracle_coeffs(0.5, 5)
    F = _dev(synth.normal_rhs(n, dim, nrhs=nrhs, tag=960 + n))
    print(f"reports: dim={dim} n={n} nrhs={nrhs} {schedule}", flush=True)
    plan = B.Plan(dim, n, weights=b.c_f64, shifts=[-x for x in b.d_f64], nrhs_max=nrhs, tol=1e-10,
                  schedule=getattr(B, "BURA_" + schedule))
    torch.cuda.synchronize()
    idle = plan.solve(F)
    G = torch.zeros_like(F)
    for _ in range(50):   # work of the caller's that the solve has to wait for
        G += F / 50
    torch.cuda.synchronize()
    G2 = torch.zeros_like(F)
    for _ in range(50):
        G2 += F / 50
    busy, again = plan.solve(G2), plan.solve(G)
    B.bura_plan_profile(plan.handle, 1)
    copied = plan.solve(F)
    assert np.array_equal(_host(idle.u), _host(copied.u))
    assert np.array_equal(_host(busy.u), _host(again.u))
    ra, rb = (np.array(list(r.report.relres)[:6]) for r in (idle, copied))
    assert np.all(np.abs(ra - rb) <= 2.0 ** -38 * rb)
    assert list(idle.report.iters)[:6] == list(copied.report.iters)[:6]
    assert abs(idle.report.err_bound - copied.report.err_bound) <= 2.0 ** -37 * copied.report.err_bound
    plan.close()
