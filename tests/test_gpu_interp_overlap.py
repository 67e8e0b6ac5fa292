"""sop_interpolate between states that share memory: the destination is
written only after the source has been read (the products along z and y go to
the workspace; a 1D destination of up to 64 points is one workgroup), zeros
outside the source box included."""
import sys

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


@pytest.mark.parametrize("na,nb,ndim,S,half", [(32, 48, 3, 2, 7.0), (48, 32, 3, 3, 5.5),
                                               (64, 64, 3, 1, 4.0), (64, 64, 1, 2, 7.0),
                                               (128, 32, 1, 1, 6.0), (32, 32, 3, 1, 3.0)])
@pytest.mark.parametrize("first", ["src", "dst"])
def test_overlapping_states(torch_cuda, na, nb, ndim, S, half, first):
    """Bitwise the result of separate buffers (the same products run)."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    ma = synth.random_small([na] * ndim, S, seed=3)
    mb = synth.random_small([nb] * ndim, S, seed=4, lo=-half, hi=half)
    pa, pb = soprop.Plan.from_model(ma, dt=0.01), soprop.Plan.from_model(mb, dt=0.01)
    psi = torch.from_numpy(synth.random_state(ma.psi0.shape, seed=9)).cuda()
    ref = torch.empty(pb.shape, dtype=torch.complex128, device="cuda")
    soprop.interpolate(pa, psi, pb, ref)
    la, lb = psi.numel(), ref.numel()
    shift = min(la, lb) // 3
    buf = torch.zeros(shift + max(la, lb) + shift, dtype=torch.complex128, device="cuda")
    oa, ob = (0, shift) if first == "src" else (shift, 0)
    a, b = buf[oa:oa + la].view(psi.shape), buf[ob:ob + lb].view(ref.shape)
    a.copy_(psi)
    soprop.interpolate(pa, a, pb, b)
    torch.cuda.synchronize()
    assert torch.equal(b, ref)
    # the rest of the source is as it was
    keep = torch.ones(buf.numel(), dtype=torch.bool, device="cuda")
    keep[ob:ob + lb] = False
    whole = torch.zeros_like(buf)
    whole[oa:oa + la] = psi.reshape(-1)
    assert torch.equal(buf[keep], whole[keep])
