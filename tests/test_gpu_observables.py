"""Observables against numpy (full FFT) on every kernel schedule: 1D of one to
1024 threads, 3D of each length, one to three surfaces, both precisions."""
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


@pytest.mark.parametrize("n,ndim,S", [(16, 1, 2), (64, 1, 1), (512, 1, 2), (1024, 1, 2),
                                      (8192, 1, 2), (32, 3, 3), (48, 3, 2), (64, 3, 1),
                                      (128, 3, 3), (256, 3, 1)])
@pytest.mark.parametrize("c64", [False, True])
def test_observables(torch_cuda, n, ndim, S, c64):
    """White-noise states, so that every frequency counts.  Tolerance: sums of
    positive terms (<V> of both signs, but of the norm's order) in FP64:
    1e-12 relative; FP32 transforms round each of log2 n stages at 6e-8: 1e-6."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([n] * ndim, S, seed=n + S)
    m.inv_mass = [0.7, 1.3, 0.4][:ndim]
    m.lo, m.hi = [-4.0, -3.0, -5.0][:ndim], [4.0, 3.5, 4.5][:ndim]
    dtype = torch.complex64 if c64 else torch.complex128
    plan = soprop.Plan.from_model(m, dt=0.01, dtype=dtype)
    psi = synth.random_state((S, *m.n), seed=4, dV=m.dV)
    if c64:
        psi = psi.astype(np.complex64).astype(complex)
    x = torch.from_numpy(psi).to(dtype).cuda()
    got = plan.observables(x)
    again = plan.observables(x)
    assert all(np.array_equal(got[k], again[k]) for k in got)  # a fixed order of sums
    assert torch.equal(x.cpu().to(torch.complex128), torch.from_numpy(psi))
    ph = np.fft.fftn(psi, axes=range(1, ndim + 1))
    p2 = (np.abs(ph) ** 2).sum(0)
    t = 0.0
    for a in range(ndim):
        k = 2 * np.pi * np.fft.fftfreq(n, m.dx[a])
        t = t + (0.5 * m.inv_mass[a] * k * k).reshape([n if b == a else 1 for b in range(ndim)])
    kin = (t * p2).sum() * m.dV / m.npts
    f = psi.reshape(S, -1)
    pops = (np.abs(f) ** 2).sum(1) * m.dV
    pot = sum((1 if i == j else 2) * (m.vtable[synth.packed_index(S, i, j)]
                                      * (f[i].conj() * f[j]).real).sum()
              for i in range(S) for j in range(i, S)) * m.dV
    tol = 1e-6 if c64 else 1e-12
    assert abs(got["kinetic"] - kin) <= tol * kin
    assert np.all(np.abs(got["pops"] - pops) <= 1e-12 * pops)
    assert abs(got["norm"] - pops.sum()) <= 1e-12 * pops.sum()
    assert abs(got["potential"] - pot) <= 1e-12 * np.abs(m.vtable).max()
    assert got["energy"] == got["kinetic"] + got["potential"]
