"""Order of a solve after the caller's pending work.

A solve waits for what is pending on its plan's stream (opts.stream), without
an event where that stream is idle.  The null stream is idle only when every
blocking stream of the device is: work on one of those comes first too.
"""

import ctypes

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture
def blocking_stream():
    """A stream that the null stream waits for (torch's own streams are not)."""
    import paper_1612_04846_amd as B
    hip = B._lib   # the library's process has the HIP runtime loaded
    create, destroy = hip.hipStreamCreate, hip.hipStreamDestroy
    create.argtypes, destroy.argtypes = [ctypes.POINTER(ctypes.c_void_p)], [ctypes.c_void_p]
    s = ctypes.c_void_p()
    assert create(ctypes.byref(s)) == 0
    yield torch.cuda.ExternalStream(s.value)
    torch.cuda.synchronize()
    assert destroy(s) == 0


@pytest.mark.parametrize("producer", ["null", "side", "blocking"])
@pytest.mark.parametrize("kind", ["const", "var"])
def test_solve_waits_for_pending_work(producer, kind, blocking_stream):
    import paper_1612_04846_amd as B
    n = 63
    F = torch.from_numpy(synth.normal_rhs(n, 2, nrhs=1, tag=1041)).cuda()
    coeff = 1.0 + 0.5 * np.random.default_rng(1).random((n + 2, n + 2)) if kind == "var" else None
    a = torch.randn(4096, 4096, device="cuda")
    side = torch.cuda.Stream()
    work = {"null": torch.cuda.default_stream(), "side": side, "blocking": blocking_stream}[producer]
    plan = B.Plan(2, n, 0.5, 7, coeff=coeff, tol=1e-10,
                  stream=side if producer == "side" else torch.cuda.default_stream())
    want = plan.solve(F).u.clone()
    f = torch.zeros_like(F)
    u = torch.empty_like(F)
    for busy in (1, 20, 0, 20):
        f.zero_()
        torch.cuda.synchronize()
        print(f"{producer} {kind}: {busy} products pending", flush=True)
        with torch.cuda.stream(work):
            b = a
            for _ in range(busy):
                b = (b @ a) * 1e-2   # milliseconds before f is there
            f.copy_(F)
        plan.solve(f, u)
        assert torch.equal(u, want)
    torch.cuda.synchronize()
    plan.close()
