"""1D runs of one, two and three steps in one call against single-step calls:
the first, middle and last piece of a run with merged step boundaries, on every
way of walking the program (held by the lanes or read by nested loops, one
surface or two, grids shorter and longer than a wave, programs longer than
what a wave holds), and the same runs as batch members."""
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


@pytest.mark.parametrize("n,S", [(16, 1), (16, 2), (32, 1), (64, 2), (128, 1), (128, 2), (256, 1),
                                 (256, 2), (512, 1), (2048, 2), (8192, 1), (8192, 2)])
@pytest.mark.parametrize("c64", [False, True])
@pytest.mark.parametrize("split,comp,order", [("VTV", "strang", 2), ("TVT", "strang", 2),
                                              ("VTV", "triple_jump", 10),
                                              ("TVT", "triple_jump", 10)])
def test_pieces(torch_cuda, n, S, c64, split, comp, order):
    """Tolerance: each of the two boundaries rounds once instead of twice, a
    few units in the last place: 1e-13 (FP64), 5e-6 (FP32).  Batch members of
    the single plan's schedule: bitwise."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([n], S, seed=5 * n + S)
    dtype = torch.complex64 if c64 else torch.complex128
    plans = [soprop.Plan.from_model(m, split=split, comp=comp, order=order, dt=0.03, dtype=dtype)
             for _ in range(3)]
    psi0 = torch.from_numpy(synth.random_state(m.psi0.shape, seed=6)).to(dtype).cuda()
    batch = soprop.Batch(plans)
    tuned = {i for f in batch.describe()["families"] if f["variant"] != 0 for i in f["members"]}
    for direction in (1, -1):
        one = psi0.clone()
        runs = []
        for steps in (1, 2, 3):
            plans[0].propagate(one, 1, direction)
            run = psi0.clone()
            plans[0].propagate(run, steps, direction)
            err = float((run - one).norm() / one.norm())
            print(f"[pieces {n} x {S} {split} {comp}{order} steps {steps}] {err:.2e}")
            assert err < (5e-6 if c64 else 1e-13)
            runs.append(run)
        members = [psi0.clone() for _ in plans]
        batch.propagate(members, [1, 2, 3], direction)
        batch.check()
        for i, (a, b) in enumerate(zip(members, runs)):
            if i in tuned:
                assert float((a - b).norm() / b.norm()) < (5e-6 if c64 else 1e-12)
            else:
                assert torch.equal(a, b)
