"""Pointer tables overwritten while the launches that read them are still queued: more pointer sets than
the plan keeps, enqueued without a wait behind work that keeps the GPU busy; every result is checked."""
import sys
import threading

import pytest
import torch

import paper_2505_10183_amd as kt

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KEPT = 8          # tables that a plan keeps on the device


@pytest.fixture(autouse=True)
def announce(request):
    print("\n[gpu-case] %s" % request.node.nodeid, file=sys.stderr, flush=True)
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("streams,stay", [(1, 0), (1, KEPT - 1), (2, 0), (2, 3)])
def test_tables_are_not_overwritten_under_queued_launches(streams, stay):
    """`stay`: calls with pointers that stay the same between those with new ones."""
    numels = [3, 4099, 17, 70001, 5]
    plan = kt.Plan(numels, "f32", 0, 16)
    n = plan.bucket_elems()[0]
    offs = [plan.tensor_info(t)[1] for t in range(len(numels))]
    sets = 4 * KEPT
    grads = [[torch.full((m,), float(100 * r + t), device=DEV) for t, m in enumerate(numels)] for r in range(sets + stay)]
    out = [torch.full((n,), -1.0, device=DEV) for _ in range(sets + stay)]
    busy = torch.randn(4096, 4096, device=DEV)
    queues = [torch.cuda.Stream() for _ in range(streams)]
    torch.cuda.synchronize()
    for q in queues:
        with torch.cuda.stream(q):
            for _ in range(20):
                busy @ busy
    for r in range(sets):
        plan.kt_bucket_pack(-1, grads[r], [out[r]], stream=queues[r % streams])
        for s in range(stay):
            plan.kt_bucket_pack(-1, grads[sets + s], [out[sets + s]], stream=queues[s % streams])
    torch.cuda.synchronize()
    for r in range(sets + stay):
        for t, m in enumerate(numels):
            assert bool((out[r][offs[t]:offs[t] + m] == float(100 * r + t)).all()), (r, t)


def test_a_table_that_grows_while_its_launch_is_queued():
    """The number of copies grows from call to call: tables are allocated anew."""
    plan = kt.Plan([5000] * 40, "f32", 5000 * 4, 16)      # 40 buckets
    nb = plan.num_buckets
    copies = [[torch.full((5000,), float(k + 1), device=DEV) for _ in range(nb)] for k in range(8)]
    busy = torch.randn(4096, 4096, device=DEV)
    outs = []
    torch.cuda.synchronize()
    for _ in range(10):
        busy @ busy
    for r in range(3 * KEPT):
        K = 1 + r // 3
        o = [torch.zeros(5000, device=DEV) for _ in range(nb)]
        plan.kt_weighted_reduce(-1, [copies[k][b] for b in range(nb) for k in range(K)], K, [1.0] * K, o)
        outs.append((K, o))
    torch.cuda.synchronize()
    for K, o in outs:
        assert all(bool((t == K * (K + 1) / 2).all()) for t in o), K


PER_THREAD = 2        # hipStreamPerThread: one handle, another stream in every thread


def test_equal_pointers_on_two_per_thread_streams():
    """Two threads call with the same pointers and with their own, each on its per-thread stream, the first
    behind work that keeps the GPU busy."""
    numels = [3, 4099, 17, 70001, 5]
    plan = kt.Plan(numels, "f32", 0, 16)
    n = plan.bucket_elems()[0]
    offs = [plan.tensor_info(t)[1] for t in range(len(numels))]
    sets = 3 * KEPT
    grads = [[torch.full((m,), float(100 * r + t), device=DEV) for t, m in enumerate(numels)] for r in range(2 * sets)]
    out = [torch.full((n,), -1.0, device=DEV) for _ in range(2 * sets)]
    both = [torch.full((n,), -1.0, device=DEV) for _ in range(KEPT // 2)]
    large = kt.Plan([1 << 25], "f32", 0, 16)
    a, b = torch.zeros(1 << 25, device=DEV), torch.zeros(large.bucket_elems()[0], device=DEV)
    torch.cuda.synchronize()

    def calls(which):
        for r in range(KEPT // 2):
            plan.kt_bucket_pack(-1, grads[r], [both[r]], stream=PER_THREAD)
        for r in range(which * sets, (which + 1) * sets):
            plan.kt_bucket_pack(-1, grads[r], [out[r]], stream=PER_THREAD)
            plan.kt_bucket_pack(-1, grads[r % (KEPT // 2)], [both[r % (KEPT // 2)]], stream=PER_THREAD)

    for _ in range(100):
        large.kt_bucket_pack(-1, [a], [b], stream=PER_THREAD)
    calls(0)
    other = threading.Thread(target=calls, args=(1,))
    other.start()
    other.join()
    torch.cuda.synchronize()
    for r, o in [*enumerate(out), *enumerate(both)]:
        for t, m in enumerate(numels):
            assert bool((o[offs[t]:offs[t] + m] == float(100 * r + t)).all()), (r, t)
