"""The backward sweep's first pass and its passes at stored steps, for every
splitting: where the boundary of two steps lies between potential actions,
after one, and between kinetic actions.  Workspaces start as NaN, so that a
value read before it is formed shows."""
import sys

import numpy as np
import pytest

from paper_1903_04946_amd import synth
from test_gpu_adjoint import base_model, sub_model

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


@pytest.mark.parametrize("surfaces", [(0, 1, 2), (0, 2), (2,)])
@pytest.mark.parametrize("split,comp,order", [("VTV", "strang", 2), ("TVT", "triple_jump", 4),
                                              ("VT", "strang", 1), ("TV", "strang", 1)])
def test_sweep_vs_oracle(torch_cuda, orc, surfaces, split, comp, order):
    """Gradient against the oracle's tangent mode, 1e-10 of the largest
    component as in the other adjoint tests, for stored steps at every, some
    and no inner boundary."""
    from paper_1903_04946_amd import soprop
    torch = torch_cuda
    S, nsteps = len(surfaces), 5
    if S == 3:
        m, theta, v0 = base_model(32)
        vt, dv, psi0 = synth.lvc_vtable_theta(m, theta), m.dvtables, m.psi0
    else:
        m, vt, dv, psi0 = sub_model(32, surfaces)
    plan = soprop.Plan(m.n, m.lo, m.hi, S, m.inv_mass, vt, split=split, comp=comp, order=order,
                       dt=10.0, dvtables=dv)
    w = np.array([0.2, -0.5, 1.0])[-S:]
    prob = orc.Problem(m.n, m.lo, m.hi, S, m.inv_mass, vt)
    sid = {"VTV": orc.VTV, "TVT": orc.TVT, "VT": orc.VT, "TV": orc.TV}[split]
    cid = {"strang": 0, "triple_jump": 1}[comp]
    opops, ograd = orc.gradient(prob, dv, psi0, sid, cid, order, 10.0, nsteps, w)
    for K in (1, 2, 3, 5, 9):
        ws = plan.adjoint_workspace(nsteps, K)
        ws.fill_(255)
        pops, grad = plan.adjoint(torch.from_numpy(psi0).cuda(), nsteps, K, w, ws)
        np.testing.assert_allclose(pops, opops, rtol=0, atol=1e-12)
        assert np.max(np.abs(grad - ograd)) < 1e-10 * max(1.0, np.max(np.abs(ograd))), K


def test_tables_of_zeros(torch_cuda):
    """A parameter whose table is zero everywhere changes nothing and has no
    gradient; the others' are those of a plan without it."""
    from paper_1903_04946_amd import soprop
    torch = torch_cuda
    m, theta, v0 = base_model(32)
    dv = np.concatenate([np.zeros_like(m.dvtables[:1]), m.dvtables])
    kw = dict(comp="triple_jump", order=4, dt=10.0)
    a = soprop.Plan(m.n, m.lo, m.hi, 3, m.inv_mass, v0, dvtables=dv, **kw)
    b = soprop.Plan(m.n, m.lo, m.hi, 3, m.inv_mass, v0, dvtables=m.dvtables, **kw)
    a.set_params(np.concatenate([[7.0], theta]))
    b.set_params(theta)
    psi0 = torch.from_numpy(m.psi0).cuda()
    got = [p.adjoint(psi0, 3, 2, [0.2, -0.5, 1.0], p.adjoint_workspace(3, 2)) for p in (a, b)]
    np.testing.assert_array_equal(got[0][0], got[1][0])
    assert got[0][1][0] == 0.0
    np.testing.assert_array_equal(got[0][1][1:], got[1][1])
    # a state of NaN has a gradient of NaN, for the zero table too
    bad = torch.full_like(psi0, float("nan"))
    assert np.isnan(a.adjoint(bad, 1, 1, [0.2, -0.5, 1.0], a.adjoint_workspace(1, 1))[1]).all()
