"""The timing hook over calls of different kinds: every kernel launch of an
observables call is bracketed, and no call is charged with the time between
it and the call before."""
import sys
import time

import numpy as np
import pytest

from paper_1903_04946_amd import synth

pytestmark = pytest.mark.gpu

GAP = 0.2  # seconds the host waits between two calls; each call takes far less


@pytest.fixture(autouse=True)
def announce(request):
    print(f"\n[gpu-case] {request.node.nodeid}", flush=True)
    sys.stdout.flush()
    yield


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1903_04946_amd import soprop
    soprop.lib()
    return torch


@pytest.mark.parametrize("n,ndim,S", [(256, 1, 2), (32, 3, 3), (48, 3, 1)])
@pytest.mark.parametrize("c64", [False, True])
def test_observables_are_timed(torch_cuda, n, ndim, S, c64):
    """3D: the three axis passes and the final sums; 1D: one kernel."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([n] * ndim, S, seed=2)
    dtype = torch.complex64 if c64 else torch.complex128
    plan = soprop.Plan.from_model(m, dt=0.01, dtype=dtype)
    psi = torch.from_numpy(m.psi0).to(dtype).cuda()
    plan.observables(psi)
    plan.set_timing(True)
    plan.observables(psi)
    kinds = plan.timing_read()
    plan.set_timing(False)
    counts = {k: v["count"] for k, v in kinds.items()}
    if ndim == 1:
        assert counts == {"other": 1}
    else:
        assert counts == {"zpass": 1, "ypass": 1, "xpass": 1, "other": 1}
        state = psi.numel() * psi.element_size()
        assert kinds["zpass"]["bytes"] == state + 8 * m.vtable.size
        assert kinds["ypass"]["bytes"] == kinds["xpass"]["bytes"] == state
    assert all(0 < v["ms"] < GAP * 1e3 for v in kinds.values())


@pytest.mark.parametrize("kind", ["trapezoid", "interpolate", "driven", "propagate", "adjoint",
                                  "observables"])
def test_no_time_between_calls(torch_cuda, kind):
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    ndim, n = (1, 512) if kind in ("trapezoid", "propagate", "driven") else (3, 32)
    m = synth.random_small([n] * ndim, 2, seed=2)
    D = synth.random_small([n] * ndim, 2, seed=3).vtable[None]
    plan = soprop.Plan.from_model(m, dt=0.01, dvtables=D)
    psi = torch.from_numpy(m.psi0).cuda()
    if kind == "interpolate":
        other = soprop.Plan.from_model(synth.random_small([n] * ndim, 2, seed=2, lo=-5, hi=5),
                                       dt=0.01)
        src = torch.from_numpy(m.psi0).cuda()
    if kind == "adjoint":
        ws = plan.adjoint_workspace(2, 1)
    call = {
        "trapezoid": lambda: plan.propagate_trapezoid(psi, 1, tol=1e-8),
        "interpolate": lambda: soprop.interpolate(other, src, plan, psi),
        "driven": lambda: plan.propagate_driven(psi, 1, f=lambda t: 0.1),
        "propagate": lambda: plan.propagate(psi, 2),
        "adjoint": lambda: plan.adjoint(psi, 2, 1, np.ones(2), ws),
        "observables": lambda: plan.observables(psi),
    }[kind]
    call()
    plan.set_timing(True)
    for _ in range(2):  # the second after untimed work and a wait of the host
        call()
        plan.observables(psi)
        plan.overlap(psi, psi)
        torch.cuda.synchronize()
        time.sleep(GAP)
    kinds = plan.timing_read()
    plan.set_timing(False)
    assert sum(v["ms"] for v in kinds.values()) < 0.5 * GAP * 1e3, kinds
