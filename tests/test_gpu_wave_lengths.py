"""Two surfaces of 256 W points on W waves against the oracle and numpy: every
W in both precisions and directions, programs longer than the 64 entries a
wave holds with merged step boundaries, batch members, and observables of the
256-point grid."""
import sys

import numpy as np
import pytest

from parity import assert_parity
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


@pytest.mark.parametrize("n", [256, 512, 1024, 2048])
@pytest.mark.parametrize("c64", [False, True])
@pytest.mark.parametrize("split,comp,order,steps", [("VTV", "triple_jump", 4, 3),
                                                    ("TVT", "triple_jump", 10, 2)])
def test_against_oracle(torch_cuda, orc, n, c64, split, comp, order, steps):
    """1e-12 in FP64 as in the other parity tests.  FP32: 5e-6 for nine substeps
    as there; over the 162 substeps of the long program the rounding's random
    walk goes sqrt(18) = 4.3 times as far, held to six times that."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([n], 2, seed=n + 7, lo=-8, hi=8)
    dtype = torch.complex64 if c64 else torch.complex128
    tol = (5e-6 if order == 4 else 3e-5) if c64 else 1e-12
    plans = [soprop.Plan.from_model(m, split=split, comp=comp, order=order, dt=0.02, dtype=dtype)
             for _ in range(2)]
    P = orc.Problem(m.n, m.lo, m.hi, m.nsurf, m.inv_mass, m.vtable, m.hbar)
    ids = ({"VTV": orc.VTV, "TVT": orc.TVT}[split], orc.TRIPLE_JUMP)
    batch = soprop.Batch(plans)
    for direction in (1, -1):
        ref = orc.propagate(P, m.psi0, *ids, order, direction * 0.02, steps)
        x = torch.from_numpy(m.psi0.copy()).to(dtype).cuda()
        plans[0].propagate(x, steps, direction)
        assert_parity(x.cpu().numpy(), ref, tol, f"{n} x 2 {split} {direction}")
        members = [torch.from_numpy(m.psi0.copy()).to(dtype).cuda() for _ in plans]
        batch.propagate(members, steps, direction)
        batch.check()
        for y in members:
            assert_parity(y.cpu().numpy(), ref, tol, f"{n} x 2 {split} {direction} member")


@pytest.mark.parametrize("n,S", [(256, 1), (256, 2), (2048, 2)])
@pytest.mark.parametrize("c64", [False, True])
def test_observables(torch_cuda, n, S, c64):
    """White noise, so that every frequency counts: 1e-12 (FP64), 1e-6 (<T> of an
    FP32 transform)."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([n], S, seed=n + S)
    dtype = torch.complex64 if c64 else torch.complex128
    plan = soprop.Plan.from_model(m, dt=0.01, dtype=dtype)
    psi = synth.random_state((S, n), seed=4, dV=m.dV)
    if c64:
        psi = psi.astype(np.complex64).astype(complex)
    got = plan.observables(torch.from_numpy(psi).to(dtype).cuda())
    k = 2 * np.pi * np.fft.fftfreq(n, m.dx[0])
    kin = (0.5 * m.inv_mass[0] * k * k * np.abs(np.fft.fft(psi, axis=1)) ** 2).sum() * m.dV / n
    pops = (np.abs(psi) ** 2).sum(1) * m.dV
    pot = sum((1 if i == j else 2) * (m.vtable[synth.packed_index(S, i, j)]
                                      * (psi[i].conj() * psi[j]).real).sum()
              for i in range(S) for j in range(i, S)) * m.dV
    assert abs(got["kinetic"] - kin) <= (1e-6 if c64 else 1e-12) * kin
    assert np.all(np.abs(got["pops"] - pops) <= 1e-12 * pops)
    assert abs(got["potential"] - pot) <= 1e-12 * np.abs(m.vtable).max()
