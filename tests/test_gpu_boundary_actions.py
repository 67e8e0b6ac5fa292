"""Step boundaries inside one call: adjoining actions of one kind run as one
action with the summed coefficient (TVT on every grid, VTV on 1D grids).  A
call of n steps against n calls of one step, which have no inner boundary."""
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


@pytest.mark.parametrize("n,ndim,S", [(16, 1, 1), (512, 1, 2), (1024, 1, 2), (4096, 1, 2),
                                      (32, 3, 3), (48, 3, 2), (128, 3, 1)])
@pytest.mark.parametrize("split,comp,order", [("TVT", "strang", 2), ("TVT", "triple_jump", 4),
                                              ("VTV", "strang", 2), ("VTV", "suzuki", 4),
                                              ("VT", "strang", 1), ("TV", "strang", 1)])
@pytest.mark.parametrize("c64", [False, True])
def test_steps_in_one_call(torch_cuda, n, ndim, S, split, comp, order, c64):
    """Tolerance: a boundary rounds once instead of twice, a few units in the
    last place of each of 7 boundaries: 1e-13 (FP64), 5e-6 (FP32)."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([n] * ndim, S, seed=3 * n + S)
    dtype = torch.complex64 if c64 else torch.complex128
    plan = soprop.Plan.from_model(m, split=split, comp=comp, order=order, dt=0.03, dtype=dtype)
    psi0 = torch.from_numpy(synth.random_state(m.psi0.shape, seed=6)).to(dtype).cuda()
    for direction in (1, -1):
        a, b, c = psi0.clone(), psi0.clone(), psi0.clone()
        plan.propagate(a, 7, direction)
        for _ in range(7):
            plan.propagate(b, 1, direction)
        plan.set_graphs(False)
        plan.propagate(c, 7, direction)
        plan.set_graphs(True)
        err = float((a - b).norm() / b.norm())
        print(f"[boundary {n}^{ndim} x {S} {split} {comp}{order} {direction}] {err:.2e}")
        assert err < (5e-6 if c64 else 1e-13)
        assert torch.equal(a, c)  # the same launches, captured or not
    if split in ("VT", "TV"):  # not reversible, and nothing adjoins
        return
    plan.propagate(a, 7, 1)  # and back
    assert float((a - psi0).norm() / psi0.norm()) < (1e-5 if c64 else 2e-13)
