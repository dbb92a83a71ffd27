"""Rounding of the FP32 preconditioner: the first iterate of a mixed plan.

With one PCG iteration and one refinement step u = alpha M f, M the multigrid
cycle; an FP64 plan with the same damping does the same in FP64, so their
difference is what FP32 rounds.  Tolerance: every step of the cycle rounds its
iterate to 2^-24 of it, and a smoother does not enlarge what came before; the
last steps that round the whole iterate, prolongation, two sweeps and the
length alpha, are four: 4 x 2^-24 (f is exact in FP32).  The sizes end in a
bottom level of one point, of 38^2 and 8^3 (which take 312 and 72 sweeps), and
have their first coarse level at 1 to 6 points per thread.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n", [(2, 63), (2, 95), (2, 127), (2, 155), (3, 15), (3, 31), (3, 35)])
@pytest.mark.parametrize("var", [False, True])
@pytest.mark.parametrize("rhs", ["normal", "ones"])
def test_fp32_cycle_rounds_like_its_steps(dim, n, var, rhs):
    import paper_1612_04846_amd as B
    rng = np.random.default_rng(7)
    shape = (1,) + (n,) * dim
    F = rng.standard_normal(shape) if rhs == "normal" else np.ones(shape)
    f = torch.from_numpy(F.astype(np.float32).astype(np.float64)).cuda()
    coeff = None
    if var:
        x = np.linspace(0.0, 1.0, n + 2)
        g = np.meshgrid(*([x] * dim), indexing="ij")
        coeff = np.exp(1.5 * np.prod([np.sin(3.0 * q + 0.4 * i) for i, q in enumerate(g)], axis=0))
    us = []
    for prec in (B.BURA_FP64, B.BURA_MIXED):
        print(f"first step: {dim}D {n} var={var} {rhs} precision {prec}", flush=True)
        plan = B.Plan(dim, n, weights=[1.0], shifts=[0.0], coeff=coeff, precision=prec, tol=1e-14, omega=0.8,
                      max_iter=1, max_outer=1)
        us.append(plan.solve(f, ok=(B.BURA_ENOCONV,)).u)
        plan.close()
    err = float((us[1] - us[0]).norm() / us[0].norm())
    print(f"  error {err * 2 ** 24:.2f} x 2^-24")
    assert err <= 4.0 * 2.0 ** -24
