"""Driven actions whose V is formed inside the z-pass: every tile, both
precisions, dense and sparse D, with and without a kinetic action after the
last potential one."""
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


@pytest.mark.parametrize("n,c64", [(n, c) for n in (32, 48, 64, 128) for c in (False, True)]
                         + [(256, False)])
@pytest.mark.parametrize("S", [2, 3])
def test_piecewise_constant_drive(torch_cuda, n, S, c64):
    """A drive constant over each step against static plans of V + s D, one
    step each (their tables come from the table kernel), to 1e-12 (FP64) and
    5e-6 (FP32) as in the other driven tests; the plan's own tables are
    untouched afterwards."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([n] * 3, S, seed=n + S)
    dtype = torch.complex64 if c64 else torch.complex128
    tol = 5e-6 if c64 else 1e-12
    D = synth.random_small([n] * 3, S, seed=7).vtable.copy()
    if S == 3:  # one coupling alone
        D[[0, 1, 2, 3, 5]] = 0.0
    base = torch.from_numpy(synth.random_state(m.psi0.shape, seed=4)).to(dtype).cuda()
    s = np.array([0.3, -1.1, 0.0])
    for split, comp, order in (("VTV", "triple_jump", 4), ("TVT", "strang", 2), ("TV", "strang", 1)):
        kw = dict(split=split, comp=comp, order=order, dt=0.02, dtype=dtype)
        plan = soprop.Plan(m.n, m.lo, m.hi, S, m.inv_mass, m.vtable, dvtables=D[None], **kw)
        got, want = base.clone(), base.clone()
        nv = len(plan.action_times())
        plan.propagate_driven(got, 3, drive=np.repeat(s[:, None], nv, axis=1))
        for si in s:
            stat = soprop.Plan(m.n, m.lo, m.hi, S, m.inv_mass, m.vtable + si * D, **kw)
            stat.propagate(want, 1)
            torch.cuda.synchronize()
        err = float((got - want).norm() / want.norm())
        print(f"[driven {n}^3 x {S} {split}] {err:.2e}")
        assert err < tol
        again, fresh = base.clone(), base.clone()
        plan.propagate(again, 2)
        soprop.Plan(m.n, m.lo, m.hi, S, m.inv_mass, m.vtable, **kw).propagate(fresh, 2)
        torch.cuda.synchronize()
        assert torch.equal(again, fresh)
