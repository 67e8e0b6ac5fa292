"""Formation of the potential's evolution operators on matrices that a smooth
model does not have: graded, degenerate, zero, huge and tiny entries, through
one potential action against numpy's eigendecomposition per point; and driven
runs whose parameter table has all or few of its entries."""
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


def _tables(kind, S, npts, rng):
    ne = S * (S + 1) // 2
    v = rng.uniform(-1.0, 1.0, (ne, npts))
    if kind == "graded":  # every entry on its own scale, down to denormal numbers
        v *= 10.0 ** rng.uniform(-320, 0, (ne, npts))
    elif kind == "degenerate":  # equal diagonals, couplings from 1 to 1e-300
        v[:] = v[0] * 10.0 ** rng.uniform(-300, 0, (ne, npts))
        for s in range(S):
            v[synth.packed_index(S, s, s)] = 0.25
    elif kind == "zero":  # zero matrices and matrices with one entry
        keep = rng.integers(0, ne + 1, npts)
        v *= (np.arange(ne)[:, None] == keep[None, :])
    elif kind == "small block":  # one large diagonal entry beside a tiny block
        v *= 1e-200
        v[0] = 1.0
    return v


@pytest.mark.parametrize("S", [2, 3])
@pytest.mark.parametrize("kind", ["graded", "degenerate", "zero", "small block", "dense"])
def test_potential_action(torch_cuda, S, kind):
    """|tau V| <= about 2 rad.  Tolerance 3e-14: about fifteen rotations of a
    few units in the last place each, in R and in R^T, and the phases'."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    rng = np.random.Generator(np.random.PCG64([S, len(kind)]))
    n = 32
    v = _tables(kind, S, n ** 3, rng)
    plan = soprop.Plan([n] * 3, [-1.0] * 3, [1.0] * 3, S, [1.0] * 3, v, dt=1.0)
    psi = synth.random_state((S, n, n, n), seed=3)
    x = torch.from_numpy(psi).cuda()
    plan.apply_action(x, "V", 1.0)
    m = np.zeros((n ** 3, S, S))
    for i in range(S):
        for j in range(S):
            m[:, i, j] = v[synth.packed_index(S, i, j)]
    lam, r = np.linalg.eigh(m)
    g = np.matmul(r.transpose(0, 2, 1), psi.reshape(S, -1).T[:, :, None])[:, :, 0]
    ref = np.matmul(r, (np.exp(-1j * lam) * g)[:, :, None])[:, :, 0].T.reshape(psi.shape)
    err = np.linalg.norm((x.cpu().numpy() - ref).ravel()) / np.linalg.norm(ref.ravel())
    print(f"[formation {kind} S={S}] rel L2 {err:.2e}")
    assert err < 3e-14


@pytest.mark.parametrize("ndim,S,entries", [(3, 3, "all"), (3, 3, "none"), (3, 2, "last"),
                                            (1, 2, "all"), (1, 1, "none")])
def test_driven_entries(torch_cuda, ndim, S, entries):
    """A constant drive s with D of all, some or no entries equals the static
    plan of V + s D.  Tolerance 1e-12, the parity bar."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([32] * ndim, S, seed=12)
    d = np.random.Generator(np.random.PCG64(5)).uniform(-0.2, 0.2, m.vtable.shape)
    if entries == "none":
        d[:] = 0.0
    elif entries == "last":
        d[:-1] = 0.0
    kw = dict(comp="triple_jump", order=4, dt=0.1)
    pd = soprop.Plan.from_model(m, dvtables=d[None], **kw)
    ps = soprop.Plan(m.n, m.lo, m.hi, S, m.inv_mass, m.vtable + 0.7 * d, **kw)
    a = torch.from_numpy(m.psi0).cuda()
    b = a.clone()
    pd.propagate_driven(a, 3, f=lambda t: 0.7)
    ps.propagate(b, 3)
    err = float((a - b).norm() / b.norm())
    print(f"[driven {ndim}D S={S} {entries}] rel L2 {err:.2e}")
    assert err < 1e-12
