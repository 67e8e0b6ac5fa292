"""Driven 1D runs and lone potential actions on every length with a body on
waves (and one without), whose last action of a step is a launch of its own,
against static plans of V + s D."""
import sys

import numpy as np
import pytest

from paper_1903_04946_amd import synth

pytestmark = pytest.mark.gpu


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


@pytest.mark.parametrize("n", [128, 256, 512, 1024, 2048])
@pytest.mark.parametrize("c64", [False, True])
def test_piecewise_constant_drive(torch_cuda, n, c64):
    """A drive constant over each step: 1e-12 (FP64) and 5e-6 (FP32), as in the
    other driven tests."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([n], 2, seed=n)
    D = synth.random_small([n], 2, seed=7).vtable
    dtype = torch.complex64 if c64 else torch.complex128
    base = torch.from_numpy(synth.random_state(m.psi0.shape, seed=4)).to(dtype).cuda()
    s = np.array([0.3, -1.1, 0.0])
    for split, comp, order in (("VTV", "triple_jump", 4), ("TVT", "strang", 2)):
        kw = dict(split=split, comp=comp, order=order, dt=0.02, dtype=dtype)
        plan = soprop.Plan(m.n, m.lo, m.hi, 2, m.inv_mass, m.vtable, dvtables=D[None], **kw)
        got, want = base.clone(), base.clone()
        plan.propagate_driven(got, 3, drive=np.repeat(s[:, None], len(plan.action_times()), axis=1))
        for si in s:
            soprop.Plan(m.n, m.lo, m.hi, 2, m.inv_mass, m.vtable + si * D, **kw).propagate(want, 1)
            torch.cuda.synchronize()
        err = float((got - want).norm() / want.norm())
        print(f"[driven {n} x 2 {split}] {err:.2e}")
        assert err < (5e-6 if c64 else 1e-12)


@pytest.mark.parametrize("n", [128, 256, 512, 1024, 2048])
@pytest.mark.parametrize("c64", [False, True])
def test_lone_potential_action(torch_cuda, n, c64):
    """exp(-i c dt V / hbar) point by point: 1e-14 (FP64) and 3e-7 (FP32: the
    state and the result rounded once each), and back again."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([n], 2, seed=n + 1)
    dtype = torch.complex64 if c64 else torch.complex128
    plan = soprop.Plan.from_model(m, dt=0.02, dtype=dtype)
    psi = synth.random_state(m.psi0.shape, seed=4)
    x = torch.from_numpy(psi).to(dtype).cuda()
    plan.apply_action(x, "V", 0.7)
    v = m.vtable
    lam, R = np.linalg.eigh(np.array([[v[0], v[1]], [v[1], v[2]]]).transpose(2, 0, 1))
    u = np.einsum("xik,xk,xjk->xij", R, np.exp(-1j * 0.7 * 0.02 * lam / m.hbar), R)
    ref = np.einsum("xij,jx->ix", u, psi)
    err = np.linalg.norm(x.cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"[lone V {n} x 2] {err:.2e}")
    assert err < (3e-7 if c64 else 1e-14)
    plan.apply_action(x, "V", -0.7)
    assert np.linalg.norm(x.cpu().numpy() - psi) / np.linalg.norm(psi) < (5e-7 if c64 else 2e-14)
