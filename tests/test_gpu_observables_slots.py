"""Where an observables call's sums go: slots of one pinned page for plans up
to its size, device memory and a copy for those beyond it, from one thread or
several, and no allocation in the first call of a plan."""
import sys
import threading
import time

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


def test_first_call_of_a_plan(torch_cuda):
    """Shortest of twenty new plans' first calls against the shortest later
    call: an allocation would be more than a call itself."""
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([256], 2, seed=3)
    psi = torch.from_numpy(m.psi0).cuda()
    first, later = [], []
    for _ in range(20):
        plan = soprop.Plan.from_model(m, dt=0.01)
        torch.cuda.synchronize()
        for times in (first, later, later):
            t = time.perf_counter()
            plan.observables(psi)
            times.append(time.perf_counter() - t)
        plan.close()
    print(f"[observables] first {min(first) * 1e6:.1f} us, later {min(later) * 1e6:.1f} us")
    assert min(first) < 1.6 * min(later)


@pytest.mark.parametrize("n,ndim,S", [(64, 1, 2), (32, 3, 3)])
def test_more_plans_than_slots(torch_cuda, n, ndim, S):
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([n] * ndim, S, seed=3)
    plans = [soprop.Plan.from_model(m, dt=0.01) for _ in range(70)]
    states = [torch.from_numpy(synth.random_state(m.psi0.shape, seed=i)).cuda() for i in range(70)]
    got = [p.observables(x) for p, x in zip(plans, states)]
    again = [p.observables(x) for p, x in zip(plans, states)]
    alone = soprop.Plan.from_model(m, dt=0.01)
    for p in plans[::2]:  # their slots are free for others
        p.close()
    ref = [alone.observables(x) for x in states]
    for a, b, c in zip(got, again, ref):
        for k in c:
            np.testing.assert_array_equal(a[k], c[k])
            np.testing.assert_array_equal(b[k], c[k])


def test_threads(torch_cuda):
    torch = torch_cuda
    from paper_1903_04946_amd import soprop
    m = synth.random_small([128], 2, seed=3)
    x = [torch.from_numpy(synth.random_state(m.psi0.shape, seed=i)).cuda() for i in range(8)]
    ref = soprop.Plan.from_model(m, dt=0.01)
    want = [ref.observables(v)["energy"] for v in x]
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        stream = torch.cuda.Stream()
        for _ in range(20):
            plan = soprop.Plan.from_model(m, dt=0.01, stream=stream)
            for _ in range(3):
                if plan.observables(x[i])["energy"] != want[i]:
                    wrong.append(i)
            plan.close()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=60)
    assert not wrong
